// Direct method on the vector ALUs: layers whose products are too few to fill matrix instructions (one or two input-side maps,
// where a chunk of eight would be padding for the most part, and small layers, which a launch without preparation serves best),
// and any shape that the matrix kernels do not take.
// Against the fp32 matrix instruction, whose launches were prepared by one that packs weights and followed by one that adds shares:
// 1 -> 4 maps of 16^3, 3^3 kernels, all three passes 39 -> 32 us; 1 -> 40 maps of 26^3, kernel gradient 23 -> 9 us.
#include <algorithm>
#include <cmath>
#include <vector>

#include "bias_parts.h"
#include "direct.h"

namespace znn {

namespace {

// Taps along x are walked in groups of U neighbours, the widest of these that divides the kernel width.
int group_width(int kx)
{
    const int widths[6] = {11, 7, 5, 4, 3, 2};
    for (int w : widths)
        if (kx % w == 0) return w;
    return 1;
}

struct FewTile {
    const float* src; const float* w; float* dst;
    int fK, fM;
    int s[3], d[3], k[3], sp[3], p[3];      // source, result, taps, tap spacing, zeros in front of the source
    long svol, dvol;
    int taps;
    long wm, wk;            // weights of result map m and source map i start at m wm + i wk
    const float* bias; float* y; const float* deriv;    // as in SplitTile
};

// A thread owns a voxel of JB result maps: a row of U taps is U loads (neighbouring lanes along x) and U JB multiply-adds with
// weights that are the same for all lanes (scalar registers).  Bound by the loads of the rows while the weights are few.
template <int U, int JB, bool BWD>
__global__ void __launch_bounds__(256) k_conv_few(FewTile P)
{
    const long v = (long)blockIdx.x * 256 + threadIdx.x;
    const int m0 = blockIdx.y * JB;
    if (v >= P.dvol) return;
    int z, y, x;
    if (P.dvol < 2147483648L) {         // uniform: 32-bit divisions where they do
        const unsigned r = (unsigned)v / (unsigned)P.d[2];
        x = (int)((unsigned)v - r * P.d[2]);
        z = (int)(r / (unsigned)P.d[1]);
        y = (int)(r - (unsigned)z * P.d[1]);
    } else {
        const long r = v / P.d[2];
        x = (int)(v - r * P.d[2]);
        z = (int)(r / P.d[1]);
        y = (int)(r - (long)z * P.d[1]);
    }
    float acc[JB];
#pragma unroll
    for (int q = 0; q < JB; ++q) acc[q] = 0.f;
    // tap t (in the order of the source, ascending) of an axis meets source coordinate x + t sp - p; it is the weight's tap
    // k - 1 - t (forward) or t (backward: reflected)
    for (int i = 0; i < P.fK; ++i) {
        const float* src = P.src + i * P.svol;
        const float* w = P.w + i * P.wk;
        for (int a = 0; a < P.k[0]; ++a) {
            const int gz = z + a * P.sp[0] - P.p[0];
            const bool okz = !BWD || (gz >= 0 && gz < P.s[0]);
            for (int b = 0; b < P.k[1]; ++b) {
                const int gy = y + b * P.sp[1] - P.p[1];
                const bool oky = okz && (!BWD || (gy >= 0 && gy < P.s[1]));
                const float* row = src + (oky ? ((long)gz * P.s[1] + gy) * P.s[2] : 0);
                const int first = BWD ? (a * P.k[1] + b) * P.k[2] : ((P.k[0] - 1 - a) * P.k[1] + P.k[1] - 1 - b) * P.k[2];
                for (int c0 = 0; c0 < P.k[2]; c0 += U) {
                    float s[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int gx = x + (c0 + u) * P.sp[2] - P.p[2];
                        const bool in = oky && (!BWD || (gx >= 0 && gx < P.s[2]));
                        const float t = row[in ? gx : 0];
                        s[u] = in ? t : 0.f;
                    }
#pragma unroll
                    for (int q = 0; q < JB; ++q) {
                        const float* wr = w + min(m0 + q, P.fM - 1) * P.wm + first + (BWD ? c0 : P.k[2] - c0 - U);     // uniform
#pragma unroll
                        for (int u = 0; u < U; ++u) acc[q] = fmaf(wr[BWD ? u : U - 1 - u], s[u], acc[q]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < JB; ++q) {
        if (m0 + q >= P.fM) return;
        const long at = (m0 + q) * P.dvol + v;
        float r = acc[q];
        if (P.deriv) r = P.deriv[at] > 0.f ? r : 0.f;       // uniform
        P.dst[at] = r;
        if (P.y) {                                          // uniform
            r += P.bias[m0 + q];
            P.y[at] = r > 0.f ? r : 0.f;
        }
    }
}

// Forward pass, four neighbouring voxels of a row by a thread (the last group of a row of at least four begins further left and repeats some of the one
// before): a load of four words takes as long as one of one, and the weights, whose latency the rows of taps wait for, serve four times as many
// products.  1 -> 40 maps, 3^3 kernels: 40^3 13.5 -> 10.4 us, 64^3 38.6 -> 19.8, 90^3 96 -> 41.
template <int U, int JB>
__global__ void __launch_bounds__(256) k_conv_few4(FewTile P)
{
    typedef float floatu4 __attribute__((ext_vector_type(4), aligned(4)));
    const unsigned groups = (unsigned)(P.d[2] + 3) / 4, v = blockIdx.x * 256 + threadIdx.x;
    const int m0 = blockIdx.y * JB;
    if (v >= groups * P.d[1] * P.d[0]) return;
    const unsigned r = v / groups;
    const int x = min((int)(v - r * groups) * 4, P.d[2] - 4), z = (int)(r / (unsigned)P.d[1]), y = (int)(r - (unsigned)z * P.d[1]);
    floatu4 acc[JB];
#pragma unroll
    for (int q = 0; q < JB; ++q) acc[q] = floatu4{0.f, 0.f, 0.f, 0.f};
    for (int i = 0; i < P.fK; ++i) {
        const float* src = P.src + i * P.svol + ((long)z * P.s[1] + y) * P.s[2] + x;
        const float* w = P.w + i * P.wk;
        for (int a = 0; a < P.k[0]; ++a)
            for (int b = 0; b < P.k[1]; ++b) {
                const float* row = src + ((long)a * P.sp[0] * P.s[1] + b * P.sp[1]) * P.s[2];
                const int first = ((P.k[0] - 1 - a) * P.k[1] + P.k[1] - 1 - b) * P.k[2];
                for (int c0 = 0; c0 < P.k[2]; c0 += U) {
                    floatu4 s[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) s[u] = *reinterpret_cast<const floatu4*>(row + (c0 + u) * P.sp[2]);
#pragma unroll
                    for (int q = 0; q < JB; ++q) {
                        const float* wr = w + min(m0 + q, P.fM - 1) * P.wm + first + P.k[2] - c0 - U;       // uniform
#pragma unroll
                        for (int u = 0; u < U; ++u)
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[q][e] = fmaf(wr[U - 1 - u], s[u][e], acc[q][e]);
                    }
                }
            }
    }
#pragma unroll
    for (int q = 0; q < JB; ++q) {
        if (m0 + q >= P.fM) return;
        const long at = (m0 + q) * P.dvol + (long)r * P.d[2] + x;
        *reinterpret_cast<floatu4*>(P.dst + at) = acc[q];
        if (P.y) {                                          // uniform
            floatu4 t;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float u = acc[q][e] + P.bias[m0 + q];
                t[e] = u > 0.f ? u : 0.f;
            }
            *reinterpret_cast<floatu4*>(P.y + at) = t;
        }
    }
}

// The same of the backward pass with neighbouring taps along x: the four voxels' rows of U taps are U + 3 loads together, of zeros outside the source.
// 40 -> 1 maps, 3^3 kernels: 38^3 15.9 -> 12.5 us, 64^3 46.7 -> 24.8; 40 -> 2, 90^3 203 -> 92; 24 -> 1, 50^3, 5^3 45.7 -> 34.1.
template <int U, int JB>
__global__ void __launch_bounds__(256) k_conv_back4(FewTile P)
{
    typedef float floatu4 __attribute__((ext_vector_type(4), aligned(4)));
    const unsigned groups = (unsigned)(P.d[2] + 3) / 4, v = blockIdx.x * 256 + threadIdx.x;
    const int m0 = blockIdx.y * JB;
    if (v >= groups * P.d[1] * P.d[0]) return;
    const unsigned r = v / groups;
    const int x = min((int)(v - r * groups) * 4, P.d[2] - 4), z = (int)(r / (unsigned)P.d[1]), y = (int)(r - (unsigned)z * P.d[1]);
    floatu4 acc[JB];
#pragma unroll
    for (int q = 0; q < JB; ++q) acc[q] = floatu4{0.f, 0.f, 0.f, 0.f};
    for (int i = 0; i < P.fK; ++i) {
        const float* src = P.src + i * P.svol;
        const float* w = P.w + i * P.wk;
        for (int a = 0; a < P.k[0]; ++a) {
            const int gz = z + a * P.sp[0] - P.p[0];
            for (int b = 0; b < P.k[1]; ++b) {
                const int gy = y + b * P.sp[1] - P.p[1];
                const bool ok = gz >= 0 && gz < P.s[0] && gy >= 0 && gy < P.s[1];
                const float* row = src + (ok ? ((long)gz * P.s[1] + gy) * P.s[2] : 0);
                for (int c0 = 0; c0 < P.k[2]; c0 += U) {
                    float s[U + 3];
#pragma unroll
                    for (int e = 0; e < U + 3; ++e) {
                        const int gx = x + c0 + e - P.p[2];
                        const bool in = ok && gx >= 0 && gx < P.s[2];
                        const float t = row[in ? gx : 0];
                        s[e] = in ? t : 0.f;
                    }
#pragma unroll
                    for (int q = 0; q < JB; ++q) {
                        const float* wr = w + min(m0 + q, P.fM - 1) * P.wm + (a * P.k[1] + b) * P.k[2] + c0;      // uniform
#pragma unroll
                        for (int u = 0; u < U; ++u)
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[q][e] = fmaf(wr[u], s[u + e], acc[q][e]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < JB; ++q) {
        if (m0 + q >= P.fM) return;
        const long at = (m0 + q) * P.dvol + (long)r * P.d[2] + x;
        if (P.deriv) {                                      // uniform
            const floatu4 d = *reinterpret_cast<const floatu4*>(P.deriv + at);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[q][e] = d[e] > 0.f ? acc[q][e] : 0.f;
        }
        *reinterpret_cast<floatu4*>(P.dst + at) = acc[q];
    }
}

using FewFn = void (*)(FewTile);

template <int U> FewFn pick_few4(int jb, bool backward)
{
    if (backward) return jb == 4 ? k_conv_back4<U, 4> : k_conv_back4<U, 8>;
    return jb == 4 ? k_conv_few4<U, 4> : k_conv_few4<U, 8>;
}

FewFn pick_few4(int u, int jb, bool backward)
{
    switch (u) {
        case 2: return pick_few4<2>(jb, backward);
        case 3: return pick_few4<3>(jb, backward);
        case 4: return pick_few4<4>(jb, backward);
        case 5: return pick_few4<5>(jb, backward);
        case 7: return pick_few4<7>(jb, backward);
        case 11: return pick_few4<11>(jb, backward);
        default: return pick_few4<1>(jb, backward);
    }
}

// Workgroups from which that is the faster way, measured at 45 to 3330: 3^3 kernels 70 of them 7.7 -> 7.3 us, 160 9.7 -> 7.8; rows of eleven taps 115 14.8 -> 18.6, 160 18.5
// -> 18.4, 200 21.8 -> 18.9, 285 25.4 -> 25.9 (a second workgroup on a few units), 440 32.9 -> 26.8, 865 57.4 -> 42.9; of seven 160 10.8 -> 9.8, 285 14.7 -> 13.8.  Backward: 3^3 kernels
// 70 8.7 -> 9.2, 160 12.3 -> 12.2; rows of eleven taps 100 19.0 -> 19.3, 160 23.6 -> 19.9, 285 32.8 -> 28.3.
constexpr long kFourGroups = 160;

template <int U> FewFn pick_few(int jb, bool backward)
{
    if (jb == 4) return backward ? k_conv_few<U, 4, true> : k_conv_few<U, 4, false>;
    return backward ? k_conv_few<U, 8, true> : k_conv_few<U, 8, false>;
}

FewFn pick_few(int u, int jb, bool backward)
{
    switch (u) {
        case 2: return pick_few<2>(jb, backward);
        case 3: return pick_few<3>(jb, backward);
        case 4: return pick_few<4>(jb, backward);
        case 5: return pick_few<5>(jb, backward);
        case 7: return pick_few<7>(jb, backward);
        case 11: return pick_few<11>(jb, backward);
        default: return pick_few<1>(jb, backward);
    }
}

// Kernel gradient: a workgroup owns U taps of one row of taps for JB output maps and one input map, and a share of the output
// voxels; a thread walks its voxels four at a time (JB + U loads and U JB multiply-adds each), and the sums of the
// threads are added in a fixed order.
struct FewGrad {
    const float* in; const float* gout; float* partial; float* gw;      // gw: written at once where there is one share
    int f, fo;
    int n[3], o[3], k[3], sp[3];
    long nvol, ovol;
    int rows, groups, jblocks;      // rows of taps, groups of U in a row, blocks of JB maps
    int shares; long span;          // voxels of a share, a multiple of 1024
};

// sum over the wave, in lane 63 (row shifts, then the rows' sums are passed on)
__device__ __forceinline__ float wave_sum(float v)
{
    auto add = [&](auto ctrl, auto rows) {
        const int t = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value, decltype(rows)::value, 0xf, true);
        v += __builtin_bit_cast(float, t);
    };
    add(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xf>{});     // row_shr:1
    add(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xf>{});
    add(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xf>{});
    add(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xf>{});
    add(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});     // row_bcast:15
    add(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});     // row_bcast:31
    return v;
}

template <int U, int JB>
__device__ __forceinline__ void grad_few(const FewGrad& P, long id, float* lds)
{
    constexpr int kAtOnce = 4;
    float (*const red)[JB * U] = reinterpret_cast<float (*)[JB * U]>(lds);      // of the four waves
    const int share = (int)(id % P.shares); id /= P.shares;
    const int cg = (int)(id % P.groups); id /= P.groups;
    const int ab = (int)(id % P.rows); id /= P.rows;
    const int jb = (int)(id % P.jblocks), i = (int)(id / P.jblocks);
    const int a = ab / P.k[1], b = ab - a * P.k[1], c0 = cg * U, j0 = jb * JB;
    // in at the shift of the group's last tap, and the taps before it sp further
    const float* in = P.in + i * P.nvol + ((long)P.sp[0] * (P.k[0] - 1 - a) * P.n[1] + P.sp[1] * (P.k[1] - 1 - b)) * P.n[2] + P.sp[2] * (P.k[2] - c0 - U);
    float acc[JB][U];
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int u = 0; u < U; ++u) acc[j][u] = 0.f;
    const long v1 = min(P.ovol, (share + 1) * P.span);
    for (long v0 = share * P.span + threadIdx.x; v0 < v1; v0 += 256 * kAtOnce) {
#pragma unroll
        for (int q = 0; q < kAtOnce; ++q) {
            const bool live = v0 + q * 256 < v1;
            const long v = live ? v0 + q * 256 : v0;
            long at;
            if (P.ovol < 2147483648L) {     // uniform
                const unsigned r = (unsigned)v / (unsigned)P.o[2], x = (unsigned)v - r * P.o[2], z = r / (unsigned)P.o[1], y = r - z * P.o[1];
                at = ((long)z * P.n[1] + y) * P.n[2] + x;
            } else {
                const long r = v / P.o[2], x = v - r * P.o[2], z = r / P.o[1], y = r - z * P.o[1];
                at = (z * P.n[1] + y) * P.n[2] + x;
            }
            float s[U], g[JB];
#pragma unroll
            for (int u = 0; u < U; ++u) s[u] = in[at + (U - 1 - u) * P.sp[2]];
#pragma unroll
            for (int j = 0; j < JB; ++j) g[j] = P.gout[min(j0 + j, P.fo - 1) * P.ovol + v];
            if (!live) {
#pragma unroll
                for (int u = 0; u < U; ++u) s[u] = 0.f;
#pragma unroll
                for (int j = 0; j < JB; ++j) g[j] = 0.f;
            }
#pragma unroll
            for (int j = 0; j < JB; ++j)
#pragma unroll
                for (int u = 0; u < U; ++u) acc[j][u] = fmaf(g[j], s[u], acc[j][u]);
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float t = wave_sum(acc[j][u]);
            if (lane == 63) red[wave][j * U + u] = t;
        }
    __syncthreads();
    const int e = threadIdx.x, j = j0 + e / U, c = c0 + e % U;
    if (e >= JB * U || j >= P.fo) return;
    const float t = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
    if (P.gw) P.gw[(((long)j * P.f + i) * P.rows + ab) * P.k[2] + c] = t;
    else P.partial[(((long)share * P.rows + ab) * P.fo + j) * ((long)P.f * P.k[2]) + (long)i * P.k[2] + c] = t;
}

template <int U, int JB>
__global__ void __launch_bounds__(256) k_grad_few(FewGrad P)
{
    __shared__ float lds[4 * JB * U];
    grad_few<U, JB>(P, blockIdx.x, lds);
}

// maps of a block where the rows of eight would have too many accumulators
constexpr bool four_only(int u) { return u >= 7; }

// Several layers with groups of U taps, and the sums of biases behind them.
constexpr int kFewItems = 8;
struct FewGrads { FewGrad item[kFewItems]; unsigned first[kFewItems]; int jb[kFewItems]; int n; unsigned bias_first; BiasItem bias[kFewBiases]; int biases; };

template <int U>
__global__ void __launch_bounds__(256) k_grads_few(FewGrads A)
{
    __shared__ float lds[4 * (four_only(U) ? 4 : 8) * U];
    if (blockIdx.x >= A.bias_first) {
        const unsigned r = blockIdx.x - A.bias_first;
        int q = 0;
        while (q + 1 < A.biases && r >= A.bias[q + 1].first) ++q;       // uniform, as below
        bias_part(A.bias[q], r - A.bias[q].first, lds);
        return;
    }
    int q = 0;
    while (q + 1 < A.n && blockIdx.x >= A.first[q + 1]) ++q;
    const long id = blockIdx.x - A.first[q];
    if constexpr (four_only(U)) grad_few<U, 4>(A.item[q], id, lds);
    else if (A.jb[q] == 4) grad_few<U, 4>(A.item[q], id, lds);
    else grad_few<U, 8>(A.item[q], id, lds);
}

using FewGradFn = void (*)(FewGrad);
using FewGradsFn = void (*)(FewGrads);

FewGradsFn pick_grads(int u)
{
    switch (u) {
        case 2: return k_grads_few<2>;
        case 3: return k_grads_few<3>;
        case 4: return k_grads_few<4>;
        case 5: return k_grads_few<5>;
        case 7: return k_grads_few<7>;
        case 11: return k_grads_few<11>;
        default: return k_grads_few<1>;
    }
}

template <int U> FewGradFn pick_grad(int jb)
{
    if constexpr (four_only(U)) return k_grad_few<U, 4>;
    else return jb == 4 ? k_grad_few<U, 4> : k_grad_few<U, 8>;
}

FewGradFn pick_grad(int u, int jb)
{
    switch (u) {
        case 2: return pick_grad<2>(jb);
        case 3: return pick_grad<3>(jb);
        case 4: return pick_grad<4>(jb);
        case 5: return pick_grad<5>(jb);
        case 7: return pick_grad<7>(jb);
        case 11: return pick_grad<11>(jb);
        default: return pick_grad<1>(jb);
    }
}

// rows of four maps where eight would leave most of them empty, or the accumulators be many
int grad_maps(const Geom& g) { return g.fo <= 4 || four_only(group_width(g.kx)) ? 4 : 8; }

long few_grad_groups(const Geom& g) { return (long)g.f * ((g.fo + grad_maps(g) - 1) / grad_maps(g)) * g.kz * g.ky * (g.kx / group_width(g.kx)); }

}  // namespace

size_t few_grad_sums_bytes(const Geom& g) { return align256((size_t)few_grad_shares(g) * g.f * g.fo * g.kvol() * sizeof(float)); }

// Shares of the voxels: four workgroups per compute unit, of no less than 4096 voxels
int few_grad_shares(const Geom& g)
{
    const long most = (g.ovol() + 4095) / 4096, want = (1024 + few_grad_groups(g) - 1) / few_grad_groups(g);
    return (int)std::max(1L, std::min(std::min(most, want), 256L));
}

// Expected seconds, from 130 layers of 1 to 40 maps and 14^3 to 64^3 voxels: the rows of taps follow each other at the latency of
// their weights (0.3 us and 0.04 us a tap), and 14e12 multiply-adds a second.  That is a thread of one voxel; with four (kFourGroups) 110 passes of large layers take 0.9 of
// it at the median, where one voxel a thread took 1.15.
double few_conv_seconds(const Geom& g, bool backward)
{
    const int U = group_width(g.kx);
    const double rows = (double)(backward ? g.fo : g.f) * g.kz * g.ky * (g.kx / U);
    const double fma = (double)g.f * g.fo * g.kvol() * (backward ? g.nvol() : g.ovol());
    return 2e-6 + rows * (0.3e-6 + 0.04e-6 * U) + fma / 14e12;
}

// From the same layers: 10e12 multiply-adds a second, and the sum of the shares where there are several.
double few_grad_seconds(const Geom& g)
{
    return 4e-6 + (double)g.f * g.fo * g.kvol() * g.ovol() / 10e12 + (few_grad_shares(g) > 1 ? 2e-6 : 0.0);
}

int few_conv(const Geom& g, bool backward, const float* src, const float* w, float* dst, const Finish& finish, hipStream_t s)
{
    FewTile P = {};
    const int n[3] = {g.nz, g.ny, g.nx}, o[3] = {g.oz, g.oy, g.ox}, k[3] = {g.kz, g.ky, g.kx}, sp[3] = {g.spz, g.spy, g.spx};
    P.src = src; P.w = w; P.dst = dst;
    P.fK = backward ? g.fo : g.f; P.fM = backward ? g.f : g.fo;
    for (int d = 0; d < 3; ++d) {
        P.s[d] = backward ? o[d] : n[d];
        P.d[d] = backward ? n[d] : o[d];
        P.k[d] = k[d]; P.sp[d] = sp[d];
        P.p[d] = backward ? sp[d] * (k[d] - 1) : 0;
    }
    P.svol = backward ? g.ovol() : g.nvol(); P.dvol = backward ? g.nvol() : g.ovol();
    P.taps = (int)g.kvol();
    P.wm = backward ? P.taps : (long)g.f * P.taps;
    P.wk = backward ? (long)g.f * P.taps : P.taps;
    P.bias = finish.bias; P.y = finish.y; P.deriv = finish.deriv;
    const int jb = P.fM <= 4 ? 4 : 8;
    const long blocks = (P.dvol + 255) / 256, groups = (P.fM + jb - 1) / jb;
    if (blocks >= 2147483647L || groups > 65535) return fail(ZNN_EUNSUPPORTED, "too many voxels or maps for one launch");
    const char* name = backward ? "direct backward (few maps)" : "direct forward (few maps)";
    const long blocks4 = ((long)P.d[0] * P.d[1] * ((P.d[2] + 3) / 4) + 255) / 256;
    // voxels that two threads take: not where the derivative is read from what is written
    const bool four = !backward || (P.sp[2] == 1 && P.deriv != P.dst);
    if (four && P.d[2] >= 4 && P.dvol < 2147483648L && blocks4 * groups >= kFourGroups)
        ZNN_LAUNCH(name, s, pick_few4(group_width(g.kx), jb, backward), dim3((unsigned)blocks4, (unsigned)groups), dim3(256), 0, P);
    else
        ZNN_LAUNCH(name, s, pick_few(group_width(g.kx), jb, backward), dim3((unsigned)blocks, (unsigned)groups), dim3(256), 0, P);
    return check_launch(name);
}

// One share: into gw (partial NULL).  Otherwise shares of partial sums in the layout of WgradSum.  The workgroups of a launch, 0: too many.
static unsigned few_grad_of(const Geom& g, const float* in, const float* gout, float* partial, float* gw, FewGrad& P, WgradSum& S)
{
    P = FewGrad{};
    const int n[3] = {g.nz, g.ny, g.nx}, o[3] = {g.oz, g.oy, g.ox}, k[3] = {g.kz, g.ky, g.kx}, sp[3] = {g.spz, g.spy, g.spx};
    P.in = in; P.gout = gout; P.partial = partial; P.gw = gw;
    P.f = g.f; P.fo = g.fo;
    for (int d = 0; d < 3; ++d) { P.n[d] = n[d]; P.o[d] = o[d]; P.k[d] = k[d]; P.sp[d] = sp[d]; }
    P.nvol = g.nvol(); P.ovol = g.ovol();
    const int U = group_width(g.kx), JB = grad_maps(g);
    P.rows = g.kz * g.ky; P.groups = g.kx / U; P.jblocks = (g.fo + JB - 1) / JB;
    P.shares = few_grad_shares(g);
    P.span = ((g.ovol() + P.shares - 1) / P.shares + 1023) / 1024 * 1024;
    P.shares = (int)((g.ovol() + P.span - 1) / P.span);
    S = WgradSum{};
    S.ksplit = P.shares; S.planes = P.rows; S.planes_b = g.ky; S.Mpad = g.fo; S.Npad = S.columns = g.f * g.kx;
    S.f = g.f; S.GA = S.GB = 1;
    for (int d = 0; d < 3; ++d) S.k[d] = k[d];
    S.slots = (long)g.fo * S.planes * S.columns;
    S.four = S.slots < 65536 && P.shares >= 16 ? 1 : 0;
    const long blocks = few_grad_groups(g) * P.shares;
    return blocks < 2147483647L ? (unsigned)blocks : 0;
}

static const char* const kFewName = "direct kernel gradient (few maps)";

int few_grad(const Geom& g, const float* in, const float* gout, float* partial, float* gw, WgradSum* sum, hipStream_t s)
{
    FewGrad P;
    const unsigned blocks = few_grad_of(g, in, gout, partial, gw, P, *sum);
    if (!blocks) return fail(ZNN_EUNSUPPORTED, "too many kernel taps for one launch");
    ZNN_LAUNCH(kFewName, s, pick_grad(group_width(g.kx), grad_maps(g)), dim3(blocks), dim3(256), 0, P);
    return check_launch(kFewName);
}

int few_grads(const GradItem* items, int count, const BiasItem* bias, int biases, unsigned bias_groups, hipStream_t s)
{
    std::vector<char> done(count, 0);
    for (int q0 = 0; q0 < count; ++q0) {
        if (done[q0]) continue;
        const int U = group_width(items[q0].g->kx);
        FewGrads A = {};
        unsigned blocks = 0;
        for (int q = q0; q < count && A.n < kFewItems; ++q) {
            const Geom& g = *items[q].g;
            if (done[q] || group_width(g.kx) != U) continue;
            const unsigned own = few_grad_of(g, items[q].in, items[q].gout, items[q].partial, nullptr, A.item[A.n], *items[q].sum);
            if (!own) return fail(ZNN_EUNSUPPORTED, "too many kernel taps for one launch");
            if (A.n && own > 2147483647u - kFewBiasGroups - blocks) break;      // the next launch's
            A.jb[A.n] = grad_maps(g);
            A.first[A.n++] = blocks;
            blocks += own;
            done[q] = 1;
        }
        A.bias_first = blocks;
        if (q0 == 0) {
            std::copy(bias, bias + biases, A.bias);
            A.biases = biases;
            blocks += bias_groups;
        }
        ZNN_LAUNCH(kFewName, s, pick_grads(U), dim3(blocks), dim3(256), 0, A);
    }
    return check_launch(kFewName);
}

}  // namespace znn
