// Direct method, forward and backward pass, on split operands as in direct_split_impl.h, for small launches: a wave has one 16-voxel tile, and four more waves of a
// workgroup bring it the halo boxes and the weights of the next chunk.
//
// Such a launch has a workgroup on a unit, or two: waves that stage in between leave its matrix cores alone meanwhile, and weights from memory, one step ahead, took 950 clocks
// a step of 290 (40 -> 40 maps, 24^3, 3^3 kernels, which the rule leaves in between: 34 000 of 44 000 clocks a workgroup; by way of LDS 16 300, as long as its reads take).
// Two buffers of each, a chunk ahead.  What is left at that size is 7 000 clocks to the first data and 7 000 of stores, which all workgroups do at once.
// Packing included, waves in between -> beside: 40 -> 40 maps, 20^3, 3^3, 17.5 -> 13.7 us forward and 21.2 -> 14.3 backward; 22 -> 7, 120 x 143, 9^2, forward 16.6 -> 11.7;
// 16 -> 24, 15^3, 3^3 two apart 9.7 -> 8.1; 7 -> 11, 15 x 24 x 41, 2 x 6 x 6, backward 13.1 -> 9.9.
//
// Tried as well: weights by LDS in several slabs of a chunk, weights straight from memory for three and four voxel tiles a wave, eight waves that multiply, five shares: 1.02 to
// 1.17 times the time of waves that stage in between.  One workgroup a unit that goes on to its next box while the four waves store the one before: 59^3 two apart
// 99 -> 110 us, the small ones 10 % slower, as registers of all phases are spent by all waves.  Results by way of LDS, stored by all waves: no gain.
#pragma once

#include "direct_split_impl.h"

namespace znn {
namespace split {

constexpr int kBesideWaves = 4;     // waves of a workgroup that multiply
constexpr int kStagers = 4;         // and those that stage

// Division by a launch constant without a branch for divisors of one: n M / 2^32 + (n & one), M as in FastDiv.
struct BoxDiv { unsigned M, one; };
inline BoxDiv make_boxdiv(unsigned d) { return BoxDiv{make_fastdiv(d).M, d <= 1 ? ~0u : 0u}; }
__device__ __forceinline__ int bdiv(int n, BoxDiv d) { return (int)(__umulhi((unsigned)n, d.M) + ((unsigned)n & d.one)); }

// In the order of use: a workgroup's way to its first load is a chain of waits for these.
struct BesideTile {
    // the workgroup's box and chunks
    int total, run;         // workgroups (boxes x sublattices), and those of one XCD
    BoxDiv dPH, dQX, dQY, dCX, dCY;     // phases, q, c (the search sees to it that all divisions are exact)
    int phases, qx, qy;     // sublattices in all, and along y and x
    int cx, cy;             // boxes per axis of a sublattice
    int Tz, Ty, Tx;         // output voxels per workgroup, on their sublattice
    int spz, spy, spx;      // tap spacing
    int nchunk, cps;        // chunks of eight input maps, and those of a share (gridDim.z shares in a launch)
    int share0;             // first share of the launch
    // LDS in bytes: one or two staging buffers, one or two of weights, tables
    int hop;                // from one staging buffer to the other (0: a single chunk)
    int wofs, whop;         // weights, and from one of their buffers to the other
    int tables;
    // staging
    int sz, sy, sx;
    int pz, py, px;         // taps of zeros virtually in front of the source (in units of the tap spacing)
    int HX, HY, hvol;       // halo box
    BoxDiv dHX, dHY;
    int fK;
    const float* src;       // K-side images [fK][sz][sy][sx]
    const uintx4* wp;       // packed weights [jgroup][chunk][step][NJ][3][64], negative where step_negative
    // walk over the taps
    int steps;              // ceil(taps / 4)
    int kz, ky, kx;
    BoxDiv dKX, dKY, dTX, dTY;
    // results
    float* dst;             // M-side images [fM][dz][dy][dx]; with several shares an array of them for each
    long share;             // elements from one share's to the next
    int fM;
    int dz, dy, dx;
    float* y;               // where not NULL: y = max(result + bias[map], 0) beside the result
    const float* bias;
    const float* deriv;     // where not NULL: the result is zero where this forward result of a rectifier is zero
    const float* w;         // weights: tap t of result map m and source map k at m wm + k wk + t, t from the end where `reflected`
    long wm, wk;
    int reflected;
};

// Workgroup barriers for data in LDS: __syncthreads() would also wait for the weights in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ void copies_barrier() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Bound by the reads of LDS, or by the latency of its ends.
template <int NJ>
__global__ void __launch_bounds__(64 * (kBesideWaves + kStagers), (kBesideWaves + kStagers) / 4) k_conv_beside(BesideTile P)
{
    constexpr int NT = 64 * kBesideWaves, NS = 64 * kStagers;       // threads that multiply, that stage
    constexpr int kStepBytes = NJ * 3 * 1024;           // packed weights of a step
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const unsigned lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, grp = lane >> 4;

    // Workgroups go to the eight XCDs in turn; each XCD takes a contiguous run, sublattices of a box next to each other:
    // they read the same cache lines.
    const int id = (blockIdx.x & 7) * P.run + (blockIdx.x >> 3);
    if (id >= P.total) return;
    const int box = bdiv(id, P.dPH), ph = id - box * P.phases;
    const int pr = bdiv(ph, P.dQX), fx = ph - pr * P.qx, fz = bdiv(pr, P.dQY), fy = pr - fz * P.qy;
    const int br = bdiv(box, P.dCX), bx = box - br * P.cx, bz = bdiv(br, P.dCY), by = br - bz * P.cy;
    // first voxel of the box
    const int z0 = fz + bz * P.Tz * P.spz, y0 = fy + by * P.Ty * P.spy, x0 = fx + bx * P.Tx * P.spx;
    const int jg = blockIdx.y;
    const int ic0 = (P.share0 + blockIdx.z) * P.cps, ic1 = min(P.nchunk, ic0 + P.cps);

    // Tables in LDS: halo offsets of the taps, four per step; packed tap (a, b, c) meets the halo at (kz-1-a, ky-1-b, kx-1-c).  And
    // the halo voxels' byte offsets in a source map, -1 outside the image (zeros).
    int* const tofs = reinterpret_cast<int*>(smem + P.tables);
    unsigned* const from = reinterpret_cast<unsigned*>(tofs + (P.steps + 2) * kTaps);

    // Four waves read, split and store the halo box of the next chunk while the others multiply, and bring them their weights.
    if (wave >= kBesideWaves) {
        const int me = threadIdx.x - NT, mine = wave - kBesideWaves;
        const long svol = (long)P.sz * P.sy * P.sx;
        const int oz = z0 - P.pz * P.spz, oy = y0 - P.py * P.spy, ox = x0 - P.px * P.spx;
        // Halo voxels r0 + me, + NS, .. of a chunk, N of them in flight; a thread stages those that it made an entry of `from` for, in the first one.
        // What `request` asks memory for goes behind its loads.
        auto stage = [&](int ic, int r0, char* buf, auto many, auto request) __attribute__((always_inline)) {
            constexpr int N = decltype(many)::value;
            const float* base = P.src + (long)ic * kMaps * svol;
            const int nvalid = P.fK - ic * kMaps;           // uniform
            const char* map[kMaps];
#pragma unroll
            for (int m = 0; m < kMaps; ++m) map[m] = reinterpret_cast<const char*>(base + min(m, nvalid - 1) * svol);
            float v[N][kMaps], scale[N];
            unsigned o[N];
            if (ic == ic0) {                                // uniform
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const int r = r0 + me + i * NS;
                    const int q = bdiv(r, P.dHX), hx = r - q * P.HX, hz = bdiv(q, P.dHY), hy = q - hz * P.HY;
                    const int gz = oz + hz * P.spz, gy = oy + hy * P.spy, gx = ox + hx * P.spx;
                    const bool in = r < P.hvol && (unsigned)gz < (unsigned)P.sz && (unsigned)gy < (unsigned)P.sy && (unsigned)gx < (unsigned)P.sx;
                    o[i] = in ? (unsigned)((gz * P.sy + gy) * P.sx + gx) * 4u : ~0u;
                    if (r < P.hvol) from[r] = o[i];
                }
            } else {
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const int r = r0 + me + i * NS;
                    o[i] = r < P.hvol ? from[r] : ~0u;
                }
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                // every load is unconditional, of some voxel of the map: a branch around each would take longer than the split
                const unsigned at = o[i] != ~0u ? o[i] : 0u;
                scale[i] = o[i] != ~0u ? kScale : 0.f;
#pragma unroll
                for (int m = 0; m < kMaps; ++m) v[i][m] = *reinterpret_cast<const float*>(map[m] + at);
            }
            request();
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int r = r0 + me + i * NS;
                if (r < P.hvol) {
                    // maps that do not exist have weights of zero
#pragma unroll
                    for (int m = 0; m < kMaps; ++m) v[i][m] *= scale[i];
                    uintx4* at = reinterpret_cast<uintx4*>(buf + r * kVoxelBytes);
#pragma unroll
                    for (int p = 0; p < 3; ++p) at[p] = take_part8(v[i]);
                }
            }
        };
        auto stage_chunk = [&](int ic, auto request) __attribute__((always_inline)) {
            char* const buf = smem + ((ic - ic0) & 1 ? P.hop : 0);
            auto nothing = [] {};
            int r0 = 0;
            for (; P.hvol - r0 > 2 * NS; r0 += 4 * NS) stage(ic, r0, buf, std::integral_constant<int, 4>{}, nothing);
            if (P.hvol - r0 > NS) stage(ic, r0, buf, std::integral_constant<int, 2>{}, request);
            else if (P.hvol > r0) stage(ic, r0, buf, std::integral_constant<int, 1>{}, request);
            else request();
        };
        global_bytes from_w = (global_bytes)(P.wp + ((long)jg * P.nchunk + ic0) * P.steps * (NJ * 3 * 64)) + lane * 16;
        for (int ic = ic0; ic < ic1; ++ic) {
            stage_chunk(ic, [&] {
                char* const to_w = smem + P.wofs + ((ic - ic0) & 1 ? P.whop : 0);
                for (int i = mine; i < P.steps * (NJ * 3); i += kStagers)
                    __builtin_amdgcn_global_load_lds((global_ptr)(from_w + i * 1024), (lds_ptr)(to_w + i * 1024), 16, 0, 0);
                from_w += P.steps * kStepBytes;
            });
            copies_barrier();                                   // the chunk is there, and the one before is no longer read
        }
        // the ends of the other waves begin with these, which come to the scalar cache meanwhile
        const BesideTile& C = *reload_args<BesideTile>();
        asm volatile("" :: "s"(C.dst), "s"(C.share), "s"(C.y), "s"(C.w));
        return;
    }

    const int taps = P.kz * P.ky * P.kx;
    {
        const int HYX = P.HY * P.HX;
        for (int t = threadIdx.x; t < (P.steps + 2) * kTaps; t += NT) {
            const int q = min(t, taps - 1);
            const int r = bdiv(q, P.dKX), c = q - r * P.kx, a = bdiv(r, P.dKY), b = r - a * P.ky;
            tofs[t] = ((P.kz - 1 - a) * HYX + (P.ky - 1 - b) * P.HX + (P.kx - 1 - c)) * kVoxelBytes;
        }
    }
    const lds_bytes lbase = (lds_bytes)smem;
    const int Ttot = P.Tz * P.Ty * P.Tx;
    int tv = wave * 16 + col;
    if (tv >= Ttot) tv = 0;
    const int vq = bdiv(tv, P.dTX), vx = tv - vq * P.Tx, vz = bdiv(vq, P.dTY), vy = vq - vz * P.Ty;
    lds_bytes voff = lbase + ((vz * P.HY + vy) * P.HX + vx) * kVoxelBytes;
    lds_bytes wl = lbase + P.wofs + lane * 16;

    // A chunk's sum is formed on its own, as by shares of one: 40 -> 40 maps, 20^3, 3^3, bit for bit what five shares gave (1.2e-7 of the largest result off 64 bits, 1.5e-7 at
    // most over six seeds); 24^3: 7.9e-8, and in one running sum 1.2e-7.
    floatx4 acc[NJ][1], sum[NJ];
    for (int ic = ic0; ic < ic1; ++ic) {
        bf16x8 a0[NJ][3], a1[NJ][3];
        uintx4 b0[3], b1[3];
        floatx4 t0[NJ], t1[NJ];
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) sum[jt] = t0[jt] = t1[jt] = floatx4{0.f, 0.f, 0.f, 0.f};
        const float lone = ic & 1 ? -1.f : 1.f;         // sign of a last step without a partner
        lds_barrier();

        lds_ints to = (lds_ints)(lbase + P.tables) + grp;
        int now = to[0], next = to[kTaps], left = P.steps;
        // q-th of the operands of a step, in the order that the products need them
        auto weight = [&](bf16x8 (&a)[NJ][3], int q) __attribute__((always_inline)) {
            const int jt = q % NJ, p = (3 - q / NJ) % 3;
            a[jt][p] = __builtin_bit_cast(bf16x8, *(lds_quads)(wl + (jt * 3 + p) * 1024));
        };
        auto voxel = [&](uintx4 (&b)[3], lds_bytes at, int q) __attribute__((always_inline)) {
            const int p = (q + 2) % 3;
            b[p] = reinterpret_cast<lds_quads>(at)[p];
        };
#pragma unroll
        for (int q = 0; q < 3 * NJ; ++q) weight(a0, q);
#pragma unroll
        for (int q = 0; q < 3; ++q) voxel(b0, voff + now, q);
        // One step: its MFMAs run while the operands of the next one arrive.  before: how add_signed takes the products of the step before, tb.
        auto step = [&](bf16x8 (&a)[NJ][3], bf16x8 (&an)[NJ][3], uintx4 (&b)[3], uintx4 (&bn)[3], floatx4 (&t)[NJ], floatx4 (&tb)[NJ],
                        auto before) __attribute__((always_inline)) {
            wl += --left > 0 ? kStepBytes : 0;          // behind the last step: that one again
            now = next;
            to += kTaps;
            next = to[kTaps];
            const lds_bytes at = voff + now;
            auto request = [&](int slot) __attribute__((always_inline)) {
                if (slot < 3) voxel(bn, at, slot);
                else if (slot < 3 + 3 * NJ) weight(an, slot - 3);
            };
            floatx4* into[NJ];
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) into[jt] = &sum[jt];
            products<NJ, decltype(before)::value, (NJ > 1)>(t, a, b, tb, lone, into, request);
        };
        const std::integral_constant<int, 1> plus;
        const std::integral_constant<int, -1> minus;
        int s = 0;
        for (; s + 2 <= P.steps; s += 2) {
            step(a0, a1, b0, b1, t0, t1, minus);
            step(a1, a0, b1, b0, t1, t0, plus);
        }
        if (s < P.steps) step(a0, a1, b0, b1, t0, t1, minus);
        const bool odd = P.steps & 1;
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) {
            add_signed<0>(sum[jt], odd ? t0[jt] : t1[jt], odd ? lone : -1.f);
            acc[jt][0] = ic == ic0 ? sum[jt] : acc[jt][0] + sum[jt];
        }
        wl += ((ic - ic0) & 1 ? -P.whop : P.whop) - (P.steps - 1) * kStepBytes;
        voff += (ic - ic0) & 1 ? -P.hop : P.hop;
    }

    bool bad = false;
#pragma unroll
    for (int jt = 0; jt < NJ; ++jt) {
        acc[jt][0] *= kUnscale;
#pragma unroll
        for (int r = 0; r < 4; ++r) bad = bad || !(fabsf(acc[jt][0][r]) <= kLargest);
    }

    const BesideTile& C = *reload_args<BesideTile>();
    const long dplane = (long)C.dy * C.dx, dvol = C.dz * dplane;
    // place of output voxel t of the box in a result map, -1 outside it
    auto voxel_of = [&](int t) -> long {
        if (t >= Ttot) return -1;
        const int q = bdiv(t, C.dTX), tx = t - q * C.Tx, tz = bdiv(q, C.dTY), ty = q - tz * C.Ty;
        const int z = z0 + tz * C.spz, y = y0 + ty * C.spy, x = x0 + tx * C.spx;
        if (z >= C.dz || y >= C.dy || x >= C.dx) return -1;
        return z * dplane + (long)y * C.dx + x;
    };
    float* const out = C.dst + blockIdx.z * C.share;
    if (C.deriv || C.y) store_tiles<NJ, 1, true>(C, acc, out, dvol, jg, wave, col, grp, voxel_of);
    else store_tiles<NJ, 1, false>(C, acc, out, dvol, jg, wave, col, grp, voxel_of);

    if (!__builtin_amdgcn_ballot_w64(bad)) return;
    auto place = [&](int t, int& tz, int& ty, int& tx) {
        const int q = bdiv(t, C.dTX);
        tx = t - q * C.Tx;
        tz = bdiv(q, C.dTY);
        ty = q - tz * C.Ty;
    };
    retake_tiles<NJ, 1>(*reload_args<BesideTile>(), out, (long)C.sz * C.sy * C.sx, dvol, jg, wave, col, grp, ic0, ic1, Ttot, taps, from, tofs, voxel_of, place);
}

}  // namespace split
}  // namespace znn
