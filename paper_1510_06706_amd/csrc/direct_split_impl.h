// Direct method, forward and backward pass, on the bf16 matrix cores at fp32 precision: kernel and the split of its
// operands.  The host side (packer, search for the workgroup's box, launch) is direct_split.hip.
//
//   D[m][n] += A[m][k] * B[k][n]      v_mfma_f32_16x16x32_bf16, six of them per product
//     m : 16 output maps              (A = packed kernel weights, coalesced 16-byte loads)
//     n : 16 output voxels            (B = input voxels read from an LDS halo box)
//     k : 8 input maps at 4 taps
//
// Layout: a workgroup of NW waves owns a box of output voxels for 16 NJ output maps; a wave owns NV of its 16-voxel tiles.
// Per chunk of eight input maps the halo box is split once and staged as [voxel][3 parts][8 maps]: an operand is one 16-byte
// LDS read, and voxels 48 bytes apart spread over the banks (3 is coprime to the 16 four-bank groups; rows of the box and the taps of
// the four lane groups still meet: 3.2 to 3.6 conflict clocks an LDS instruction, a tenth of the time).  A lane group of 16
// reads its own tap of the step's four, at an offset it looks up once per step, so the walk over the taps is the same for
// every kernel shape; the count is padded to a multiple of four with weights of zero.
//
// Measured against v_mfma_f32_16x16x4_f32 on 4-map chunks of the same halo boxes, forward / backward pass: 40 -> 40 maps, 64^3, 5^3 kernels 740 /
// 780 -> 500 / 475 us (173, 182 TFLOP/s of fp32 products); 80 -> 80, 256^2, 11^2: 806 / 741 -> 435 / 432 us; 120 -> 120, 48^3, 7^3:
// 9.2 / 9.0 -> 3.3 / 4.4 ms; 40 -> 40, 24^3, 3^3: 32 / 39 -> 22 / 23 us; the same, 60^3, taps two apart: 227 / 213 -> 98 /
// 131 us.  Error against 64 bits (2-norm) of the same layers: 9.1e-7 -> 2.5e-7, 1.2e-6 -> 3.3e-7, 2.6e-6 -> 6.7e-7,
// 1.6e-7 -> 8.8e-8, 4.2e-7 -> 1.2e-7: sums of a step on their own are what does it (kept in one running sum, the six
// instructions would be as far off as the fp32 one).
//
// Sparse taps (s voxels apart) tie together only voxels of the same residues modulo s: a workgroup's box lies on one of the
// s_z s_y s_x sublattices, on which the taps are neighbours, so the halo of a sparse layer is that of a dense one.
#pragma once

#include <type_traits>

#include "split_parts.h"

namespace znn {
namespace split {

constexpr int kMaps = 8;            // input maps of a chunk
constexpr int kTaps = 4;            // taps of a step
constexpr int kVoxelBytes = kVectorBytes;     // three parts of eight maps
constexpr int kFetch = 2;           // halo voxels a thread has in flight

// Sign of a step: every second one of a chunk, and a last one without a partner in every second chunk.
__device__ __forceinline__ bool step_negative(int step, int steps, int chunk)
{
    return step & 1 || ((steps & 1) && step == steps - 1 && (chunk & 1));
}

struct SplitTile {
    const float* src;       // K-side images [fK][sz][sy][sx]
    const uintx4* wp;       // packed weights [jgroup][chunk][step][NJ][3][64], negative where step_negative
    float* dst;             // M-side images [fM][dz][dy][dx]
    const float* w;         // weights: tap t of result map m and source map k at m wm + k wk + t, t from the end where `reflected`
    long wm, wk;
    int reflected;
    int fK, fM;
    int sz, sy, sx;
    int pz, py, px;         // taps of zeros virtually in front of the source (in units of the tap spacing)
    int dz, dy, dx;
    int kz, ky, kx;
    int spz, spy, spx;      // tap spacing
    int Tz, Ty, Tx;         // output voxels per workgroup, on their sublattice
    int HZ, HY, HX, hvol;   // halo box
    int cy, cx;             // boxes per axis of a sublattice
    int qy, qx, phases;     // sublattices along y and x, and in all
    int total, run;         // workgroups (boxes x sublattices), and those of one XCD
    int nchunk, cps;        // chunks of eight input maps, and those of a share (gridDim.z shares in a launch)
    int share0;             // first share of the launch
    int steps;              // ceil(taps / 4)
    float* partial;         // [shares][fM][dz][dy][dx] where gridDim.z > 1
    float* y;               // where not NULL: y = max(result + bias[map], 0) beside the result
    const float* bias;
    const float* deriv;     // where not NULL: the result is zero where this forward result of a rectifier is zero
    FastDiv dHX, dHY, dTX, dTY, dKX, dKY, dPH, dQX, dQY, dCX, dCY;      // H, T, k, phases, q, c (the search sees to it that they are exact)
};

using SplitFn = void (*)(SplitTile);

// The launch's parameters from memory again: those of the end of a workgroup need not stay in scalar registers from its beginning on.
template <class Args>
__device__ __forceinline__ const Args* reload_args()
{
    auto args = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    return (const Args*)args;
}

// Stores what the accumulators hold.  Lane holds maps 4 (lane / 16) + r of voxel lane % 16.  A result's place is that of the lane's first map plus a uniform step, and the
// derivatives of a voxel tile are loaded together: with a 64-bit product for each place, and each derivative waited for before the next, the stores of
// a workgroup took 11 000 clocks (now 4200; 12 -> 8 us a launch on the last layer of a net).
template <int NJ, int NV, bool FINISH, class Args, class VoxelOf>
__device__ __forceinline__ void store_tiles(const Args& C, const floatx4 (&acc)[NJ][NV], float* out, long dvol, int jg, int wave, int col, int grp, VoxelOf voxel_of)
{
    float bias[NJ][4];
    if (FINISH && C.y) {                            // uniform
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
            for (int r = 0; r < 4; ++r) bias[jt][r] = C.bias[min((jg * NJ + jt) * 16 + grp * 4 + r, C.fM - 1)];
    }
#pragma unroll
    for (int nv = 0; nv < NV; ++nv) {
        const long vox = voxel_of((wave * NV + nv) * 16 + col);
        if (vox < 0) continue;
        const long first = (jg * NJ * 16 + grp * 4) * dvol + vox;
        float v[NJ][4], d[NJ][4];
        if (FINISH && C.deriv) {                    // uniform; all loads are in flight together
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    d[jt][r] = C.deriv[(jg * NJ + jt) * 16 + grp * 4 + r < C.fM ? first + (jt * 16 + r) * dvol : vox];
        }
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) {
            const int left = C.fM - (jg * NJ + jt) * 16;            // maps of the tile (uniform)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[jt][r] = acc[jt][nv][r];
                if (FINISH && C.deriv) v[jt][r] = d[jt][r] > 0.f ? v[jt][r] : 0.f;
                if (left >= 16 || grp * 4 + r < left) {
                    float* const at = out + first + (jt * 16 + r) * dvol;
                    *at = v[jt][r];
                    if (FINISH && C.y) {
                        const float u = v[jt][r] + bias[jt][r];
                        C.y[first + (jt * 16 + r) * dvol] = u > 0.f ? u : 0.f;
                    }
                }
            }
        }
    }
}

// An infinity or a NaN among the operands (or the voxel read in place of a zero) makes the parts' products NaN where the
// product itself may not be: results that are not finite are read back and taken again in fp32, straight from memory, on
// v_mfma_f32_16x16x4_f32, a voxel tile at a time.  A NaN stays one, so a tile is done when all of these are; the finite ones stand.
// 40 -> 40 maps, 64^3, 5^3 kernels, forward 560 us on finite values: weights of half the maps NaN 480 us (6.0 ms where a wave took all
// of its tiles again), all voxels NaN 510, one voxel infinite 800; 80 -> 80, 256^2, 11^2, 430 us: 400, 400 and 2900 us.
template <int NJ, int NV, class Args, class VoxelOf, class Place>
__device__ __forceinline__ void retake_tiles(const Args& C, float* out, long svol, long dvol, int jg, int wave, int col, int grp, int ic0, int ic1, int Ttot, int taps,
                                             const unsigned* from, const int* tofs, VoxelOf voxel_of, Place place)
{
    const int maps = min(ic1 * kMaps, C.fK);
#pragma unroll 1
    for (int nv = 0; nv < NV; ++nv) {
        const int t = (wave * NV + nv) * 16 + col;
        const long vox = voxel_of(t);
        int tz, ty, tx;
        place(t < Ttot ? t : 0, tz, ty, tx);
        const unsigned* const at = from + (tz * C.HY + ty) * C.HX + tx;
        unsigned wrong = 0;                                     // the lane's results that are
        floatx4 again[NJ];
        global_floats row[NJ];                                  // weights of the lane's result map (or the last one, for no result)
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) {
            again[jt] = floatx4{0.f, 0.f, 0.f, 0.f};
            row[jt] = (global_floats)C.w + min((jg * NJ + jt) * 16 + (int)col, C.fM - 1) * C.wm;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = (jg * NJ + jt) * 16 + grp * 4 + r;
                if (vox >= 0 && j < C.fM && !(fabsf(out[(long)j * dvol + vox]) <= kLargest)) wrong |= 1u << (jt * 4 + r);
            }
        }
        // whether some of them are not NaN again yet
        auto open = [&] {
            unsigned left = wrong;
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (again[jt][r] != again[jt][r]) left &= ~(1u << (jt * 4 + r));
            return __builtin_amdgcn_ballot_w64(left != 0) != 0;
        };
        // Products of `N` input maps at taps t0 to t0 + 15, N of its four by a lane: a result map's weights of these are 64 contiguous bytes.
        auto add_products = [&](int map, int t0, auto many) {
            constexpr int N = decltype(many)::value;
            float v[N][N], w[N][N][NJ];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int q = t0 + 4 * grp + i, tap = min(q, taps - 1);
                const unsigned o = q < taps ? at[tofs[tap] / kVoxelBytes] : ~0u;
#pragma unroll
                for (int h = 0; h < N; ++h) {
                    const long of = min(map + h, maps - 1);         // uniform
                    const bool has = q < taps && map + h < maps;
                    const float x = ((global_floats)C.src + of * svol)[o != ~0u ? o / 4 : 0];
                    v[i][h] = has && o != ~0u ? x : 0.f;
#pragma unroll
                    for (int jt = 0; jt < NJ; ++jt) {
                        const float y = row[jt][of * C.wk + (C.reflected ? taps - 1 - tap : tap)];
                        w[i][h][jt] = has ? y : 0.f;
                    }
                }
            }
#pragma unroll
            for (int h = 0; h < N; ++h)
#pragma unroll
                for (int i = 0; i < N; ++i)
#pragma unroll
                    for (int jt = 0; jt < NJ; ++jt) again[jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i][h][jt], v[i][h], again[jt], 0, 0, 0);
        };
        // Where a few products make NaN of them already, no more are needed: whole maps of a net that has diverged.  The walk is bound by
        // the way to memory, so a step of it requests much.
        bool more = open();
        if (more) {
            add_products(ic0 * kMaps, 0, std::integral_constant<int, 1>{});
            more = open();
        }
        if (more) {
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) again[jt] = floatx4{0.f, 0.f, 0.f, 0.f};
            for (int map = ic0 * kMaps; map < maps && more; map += 4)
                for (int t0 = 0; t0 < taps && more; t0 += 16) {
                    add_products(map, t0, std::integral_constant<int, 4>{});
                    more = open();
                }
        }
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (wrong >> (jt * 4 + r) & 1) {
                    const int j = (jg * NJ + jt) * 16 + grp * 4 + r;
                    const long to = (long)j * dvol + vox;
                    float s = again[jt][r];
                    out[to] = s;
                    if (C.y) {                                          // uniform
                        s += C.bias[j];
                        C.y[to] = s > 0.f ? s : 0.f;
                    }
                }
    }
}

// Bound by the matrix cores (six MFMAs of 16 clocks per 16 x 16 x 32 product).
// Two waves on a SIMD, by registers; four of 2 x 2 tiles, which are one over that by themselves.
template <int NJ, int NV, int NW>
__global__ void __launch_bounds__(64 * NW, NJ == 2 && NV == 2 ? 4 : 2) k_conv_split(SplitTile P)
{
    constexpr int NT = 64 * NW;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const unsigned lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, grp = lane >> 4;

    // Workgroups go to the eight XCDs in turn; each XCD takes a contiguous run, sublattices of a box next to each other:
    // they read the same cache lines.
    const int id = (blockIdx.x & 7) * P.run + (blockIdx.x >> 3);
    if (id >= P.total) return;
    const int box = (int)fdiv((unsigned)id, P.dPH), ph = id - box * P.phases;
    const int pr = (int)fdiv((unsigned)ph, P.dQX), fx = ph - pr * P.qx, fz = (int)fdiv((unsigned)pr, P.dQY), fy = pr - fz * P.qy;
    const int br = (int)fdiv((unsigned)box, P.dCX), bx = box - br * P.cx, bz = (int)fdiv((unsigned)br, P.dCY), by = br - bz * P.cy;
    const int z0 = bz * P.Tz, y0 = by * P.Ty, x0 = bx * P.Tx;       // on the sublattice
    const int Ttot = P.Tz * P.Ty * P.Tx;
    const long splane = (long)P.sy * P.sx, svol = P.sz * splane;
    const long dplane = (long)P.dy * P.dx, dvol = P.dz * dplane;
    const int jg = blockIdx.y;
    const int ic0 = (P.share0 + blockIdx.z) * P.cps, ic1 = min(P.nchunk, ic0 + P.cps);

    auto place = [&](int t, int& tz, int& ty, int& tx) {
        const int q = (int)fdiv((unsigned)t, P.dTX);
        tx = t - q * P.Tx;
        tz = (int)fdiv((unsigned)q, P.dTY);
        ty = q - tz * P.Ty;
    };
    // place of output voxel t of the box in a result map, -1 outside it
    auto voxel_of = [&](int t) -> long {
        if (t >= Ttot) return -1;
        int tz, ty, tx;
        place(t, tz, ty, tx);
        const int z = fz + (z0 + tz) * P.spz, y = fy + (y0 + ty) * P.spy, x = fx + (x0 + tx) * P.spx;
        if (z >= P.dz || y >= P.dy || x >= P.dx) return -1;
        return z * dplane + (long)y * P.dx + x;
    };

    // halo offsets of the taps, four per step; packed tap (a, b, c) meets the halo at (kz-1-a, ky-1-b, kx-1-c)
    int* const tofs = reinterpret_cast<int*>(smem + P.hvol * kVoxelBytes);
    const int taps = P.kz * P.ky * P.kx;
    for (int t = threadIdx.x; t < (P.steps + 2) * kTaps; t += NT) {
        const int q = min(t, taps - 1);
        const int r = (int)fdiv((unsigned)q, P.dKX), c = q - r * P.kx, a = (int)fdiv((unsigned)r, P.dKY), b = r - a * P.ky;
        tofs[t] = (((P.kz - 1 - a) * P.HY + (P.ky - 1 - b)) * P.HX + (P.kx - 1 - c)) * kVoxelBytes;
    }
    // halo voxels: byte offset in a source map, -1 outside the image (zeros)
    unsigned* const from = reinterpret_cast<unsigned*>(tofs + (P.steps + 2) * kTaps);
    for (int r = threadIdx.x; r < P.hvol; r += NT) {
        const int r1 = (int)fdiv((unsigned)r, P.dHX), hx = r - r1 * P.HX;
        const int hz = (int)fdiv((unsigned)r1, P.dHY), hy = r1 - hz * P.HY;
        const int gz = fz + (z0 + hz - P.pz) * P.spz, gy = fy + (y0 + hy - P.py) * P.spy, gx = fx + (x0 + hx - P.px) * P.spx;
        const bool in = gz >= 0 && gz < P.sz && gy >= 0 && gy < P.sy && gx >= 0 && gx < P.sx;
        from[r] = in ? (unsigned)((gz * P.sy + gy) * P.sx + gx) * 4u : ~0u;
    }
    const lds_bytes lbase = (lds_bytes)smem;
    lds_bytes voff[NV];
#pragma unroll
    for (int nv = 0; nv < NV; ++nv) {
        int t = (wave * NV + nv) * 16 + col;
        if (t >= Ttot) t = 0;
        int tz, ty, tx;
        place(t, tz, ty, tx);
        voff[nv] = lbase + ((tz * P.HY + ty) * P.HX + tx) * kVoxelBytes;
    }

    floatx4 acc[NJ][NV];
#pragma unroll
    for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
        for (int nv = 0; nv < NV; ++nv) acc[jt][nv] = floatx4{0.f, 0.f, 0.f, 0.f};

    // A thread reads, splits and stores the halo voxels it has an entry of `from` for, so this needs no barrier before it.
    // Its latency is left to the other workgroup of the compute unit: loads kept in flight through the taps would take the
    // registers of two result tiles.
    auto stage = [&](int ic) {
        const float* base = P.src + (long)ic * kMaps * svol;
        const int nvalid = P.fK - ic * kMaps;           // uniform
        const char* map[kMaps];
#pragma unroll
        for (int m = 0; m < kMaps; ++m) map[m] = reinterpret_cast<const char*>(base + min(m, nvalid - 1) * svol);
        for (int r0 = threadIdx.x; r0 < P.hvol; r0 += kFetch * NT) {
            float v[kFetch][kMaps];
#pragma unroll
            for (int i = 0; i < kFetch; ++i) {
                const int r = r0 + i * NT;
                // every load is unconditional, of some voxel of the map: a branch around each would take longer than the split
                const unsigned o = r < P.hvol ? from[r] : ~0u, at = o != ~0u ? o : 0u;
#pragma unroll
                for (int m = 0; m < kMaps; ++m) v[i][m] = *reinterpret_cast<const float*>(map[m] + at);
            }
#pragma unroll
            for (int i = 0; i < kFetch; ++i)
                if (r0 + i * NT < P.hvol) {
                    // maps that do not exist have weights of zero
                    const float scale = from[r0 + i * NT] != ~0u ? kScale : 0.f;
#pragma unroll
                    for (int m = 0; m < kMaps; ++m) v[i][m] *= scale;
                    uintx4* at = reinterpret_cast<uintx4*>(smem + (r0 + i * NT) * kVoxelBytes);
#pragma unroll
                    for (int p = 0; p < 3; ++p) at[p] = take_part8(v[i]);
                }
        }
    };

    // Few tiles wait for their weights, all of a step's at once before its products are the earliest (29 -> 7 maps, 12^3, 7^3, backward, 2 x 1: 25.1 us, paced 29.8; 36 passes of
    // 5 x 1 tiles: paced 1.005 of the time, to 1.05); the largest tile shapes have no registers for it.
    constexpr bool LARGE = NJ * NV == 18 || (NJ == 5 && NV == 2);
    constexpr bool PACED = NJ > 1 && NJ * NV > 5 && !LARGE;
    // Packed weights: a uniform place and the lane's offset, or the lane's place alone.  By that 2 x 2 tiles keep to the registers of four waves, 5 x 2 tiles take 0.992 of the
    // time (44 passes) and 2 x 1 tiles 0.979 (40 passes; 17 -> 17 maps, 16 x 10 x 11, 7^3, backward, 29.1 -> 28.2 us).
    constexpr bool UNIFORM = (NJ != 2 || NV > 2) && (NJ != 5 || NV != 2);
    global_bytes wq = (global_bytes)(P.wp + ((long)jg * P.nchunk + ic0) * P.steps * (NJ * 3 * 64)) + (UNIFORM ? 0 : lane * 16);
    const unsigned wlane = UNIFORM ? lane * 16 : 0;
    for (int ic = ic0; ic < ic1; ++ic) {
        bf16x8 a0[NJ][3], a1[NJ][3];
        uintx4 b0[3], b1[3];
        floatx4 t0[NJ], t1[NJ];
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) t0[jt] = t1[jt] = floatx4{0.f, 0.f, 0.f, 0.f};
        // q-th of the operands of a step, paced in the order that the products need them
        auto weight = [&](bf16x8 (&a)[NJ][3], int q) __attribute__((always_inline)) {
            const int jt = PACED ? q % NJ : q / 3, p = PACED ? (3 - q / NJ) % 3 : q % 3;
            a[jt][p] = __builtin_bit_cast(bf16x8, *(global_quads)(wq + (jt * 3 + p) * 1024 + wlane));
        };
#pragma unroll
        for (int q = 0; q < 3 * NJ; ++q) weight(a0, q);
        const float lone = ic & 1 ? -1.f : 1.f;         // sign of a last step without a partner
        __syncthreads();                                // nobody still reads the chunk before
        stage(ic);
        __syncthreads();

        lds_ints to = (lds_ints)(lbase + P.hvol * kVoxelBytes) + grp;
        int now = to[0], next = to[kTaps];
        auto voxel = [&](uintx4 (&b)[3], lds_bytes at, int q) __attribute__((always_inline)) {
            const int p = PACED ? (q + 2) % 3 : q;
            b[p] = reinterpret_cast<lds_quads>(at)[p];
        };
#pragma unroll
        for (int q = 0; q < 3; ++q) voxel(b0, voff[0] + now, q);
        // One step: the MFMAs of a voxel tile run while the operands of the next one arrive.  PAR: which register set of
        // the voxel operands the step's first tile is in; sign, before: how add_signed takes its tiles, and those before.
        auto step = [&](bf16x8 (&a)[NJ][3], bf16x8 (&an)[NJ][3], auto sign, auto before, auto par) __attribute__((always_inline)) {
            constexpr int PAR = decltype(par)::value;
            wq += NJ * 3 * 1024;                        // behind the last step: the next chunk's, or the padding
            if constexpr (UNIFORM) asm volatile("" : "+s"(wq));     // a uniform place it stays
#pragma unroll
            for (int nv = 0; nv < NV; ++nv) {
                uintx4 (&b)[3] = ((PAR + nv) & 1) ? b1 : b0;
                uintx4 (&bn)[3] = ((PAR + nv) & 1) ? b0 : b1;
                if (nv + 1 == NV) {
                    now = next;
                    to += kTaps;
                    next = to[kTaps];
                }
                const lds_bytes at = voff[(nv + 1) % NV] + now;
                auto request = [&](int slot) __attribute__((always_inline)) {
                    if constexpr (!PACED) {
                        if (nv == 0 && slot < 3 * NJ) weight(an, slot);
                        if (slot >= 3 * NJ && slot < 3 * NJ + 3) voxel(bn, at, slot - 3 * NJ);
                        return;
                    }
                    if (slot < 3) voxel(bn, at, slot);
                    // behind them the weights, but for those of few tiles, which have to come from memory in their time
                    constexpr int WAIT = NJ * NV <= 6 ? 0 : 3;
                    const int q = nv * (6 * NJ - WAIT) + slot - WAIT;
                    if (q < 3 * NJ && slot >= WAIT) weight(an, q);
                };
                floatx4* into[NJ];
#pragma unroll
                for (int jt = 0; jt < NJ; ++jt) into[jt] = &acc[jt][(nv + NV - 1) % NV];
                floatx4 (&t)[NJ] = (PAR + nv) & 1 ? t1 : t0;
                floatx4 (&tb)[NJ] = (PAR + nv) & 1 ? t0 : t1;       // the tile before; for the first one, of the step before
                if (nv == 0) products<NJ, decltype(before)::value, PACED>(t, a, b, tb, lone, into, request);
                else products<NJ, decltype(sign)::value, PACED>(t, a, b, tb, lone, into, request);
            }
        };
        constexpr int ODD = NV & 1;
        const std::integral_constant<int, 1> plus;
        const std::integral_constant<int, -1> minus;
        const std::integral_constant<int, 0> either;
        int s = 0;
        for (; s + 2 <= P.steps; s += 2) {
            step(a0, a1, plus, minus, std::integral_constant<int, 0>{});
            step(a1, a0, minus, plus, std::integral_constant<int, ODD>{});
        }
        if (s < P.steps) step(a0, a1, either, minus, std::integral_constant<int, 0>{});
        // the last tile's: in set 0 or 1 by the parity of steps x NV
        const float last = P.steps & 1 ? lone : -1.f;
        if (P.steps & ODD & 1) {
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) add_signed<0>(acc[jt][NV - 1], t0[jt], last);
        } else {
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) add_signed<0>(acc[jt][NV - 1], t1[jt], last);
        }
    }

#pragma unroll
    for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
        for (int nv = 0; nv < NV; ++nv) acc[jt][nv] *= kUnscale;

    bool bad = false;
#pragma unroll
    for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
        for (int nv = 0; nv < NV; ++nv)
#pragma unroll
            for (int r = 0; r < 4; ++r) bad = bad || !(fabsf(acc[jt][nv][r]) <= kLargest);

    // The largest tile shapes work out the places of their voxels again, from the thread's number: kept from the start these went to memory (3 x 6 tiles four registers,
    // now none; 5 x 2 tiles six, now two).  44 passes each: 0.989 and 0.992 of the time.  Others have registers left for them.
    unsigned thread = threadIdx.x;
    if constexpr (LARGE) asm volatile("" : "+v"(thread));
    const int ecol = thread & 15, egrp = thread >> 4 & 3;
    float* const out = gridDim.z > 1 ? P.partial + (long)blockIdx.z * P.fM * dvol : P.dst;
    // what follows the sums is decided once, outside the stores
    if (P.deriv || P.y) store_tiles<NJ, NV, true>(P, acc, out, dvol, jg, wave, ecol, egrp, voxel_of);
    else store_tiles<NJ, NV, false>(P, acc, out, dvol, jg, wave, ecol, egrp, voxel_of);

    if (!__builtin_amdgcn_ballot_w64(bad)) return;
    retake_tiles<NJ, NV>(*reload_args<SplitTile>(), out, svol, dvol, jg, wave, ecol, egrp, ic0, ic1, Ttot, taps, from, tofs, voxel_of, place);
}

}  // namespace split
}  // namespace znn
