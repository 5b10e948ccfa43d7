// Kernel gradient of the direct method on the bf16 matrix cores at fp32 precision (split_parts.h).
//
//   gw[j][i][tap] = sum_v gout[j][v] * in[i][v + shift(tap)]      shift = s (k - 1 - tap)
//
// is a product D[m][n] += A[m][k] B[k][n] whose reduction runs over the output voxels:
//     m : 16 output maps                        (A = gout)
//     n : 16 of the columns (input map, tap)    (B = in, shifted)
//     k : 4 neighbouring places of x times a vector of 8 voxels
//
// The eight voxels of a vector lie Q apart, not next to each other: every axis is cut into E_d equal pieces of Q_d (E_z E_y
// E_x = 8) and voxel q of all eight pieces makes vector q.  A shift by a tap is then a shift of vectors on every axis, so
// operands of all taps are aligned 16-byte reads.  With sparse taps (s voxels apart) an axis falls into its s residues
// first, which no tap ties together, and each is cut into pieces.  k_split_images writes both images in that order, split, once
// per call: gout with zeros behind its pieces, in with the k - 1 vectors behind each piece that belong to the next one.
//
// A workgroup of eight waves owns a group of taps (GA planes, GB rows of each, all along x) and of columns, all rows of NJ map
// tiles, and a share of the tiles of Rz x Ry x TX vectors; a tile and its halo travel global -> LDS (16 bytes per lane, no
// registers) into one of two buffers while the other is used.  The waves form NG sets with NT column tiles each, the KW waves of
// a set take every KW-th step of a tile, and their sums are added at the end.  The partial sums of the shares are
// added by a second kernel in ascending order.
//
// Measured against v_mfma_f32_16x16x4_f32 on rows of the images as they are, launches of a call together: 40 -> 40 maps, 64^3, 5^3
// kernels 960 -> 538 us (161 TFLOP/s of fp32 products); 80 -> 80, 256^2, 11^2: 970 -> 495 us; 24 -> 36, 23 x 75 x 61,
// 3 x 5 x 5: 223 -> 122 us (rows of odd lengths had 4-byte copies); 120 -> 120, 48^3, 7^3: 9.7 -> 4.2 ms; 40 -> 40, 24^3,
// 3^3: 36 -> 32 us.  Matrix cores busy 0.55 of the first one's time: the waves of a workgroup begin every step of a
// tile with its operands, and 3.9 conflict clocks an LDS instruction are a tenth of the time.  Two workgroups of four waves per compute unit, each with half the buffers, would overlap these, but their smaller
// tiles are copied more often: 542 -> 887 us.
#pragma once

#include "split_parts.h"

namespace znn {
namespace split {

typedef __attribute__((address_space(1))) const void* global_cptr;
typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr int kGradWaves = 8;
constexpr int kGradBuffer = 78 * 1024;      // bytes of a tile buffer
constexpr int kGradSpans = 10;              // copies of 1 KiB of a tile per wave

struct GradTile {
    const uintx4* gs;       // gout, split: [fo][PZ][PY][PX][3], negative in every second step
    const uintx4* is;       // in, split: [f][IZ][IY][IX][3]
    const float* in; const float* gout; float* partial;
    int f, fo;
    int n[3], o[3], k[3], sp[3];
    int E[3], Q[3];         // pieces of a residue per axis, voxels of a piece
    int P[3], I[3];         // vectors per axis of gs and is, all residues
    int T[3];               // tiles of a residue per axis; tile t of an axis is one of residue t / T
    int r0[3], q0[3];       // residue and vector of a residue that gs and is begin with
    int more;               // 1: the sums are added to what `partial` holds of earlier launches
    int R[3], H[3];         // vectors of a tile, and of its halo box in `is`
    int GA, GB, planes_b;   // tap planes and rows of a group, groups along y
    int GS, IS;             // bytes of a map in LDS (gout, in)
    int tiles_y, tiles_x, tiles, tps;   // tiles of all residues per axis and in all, tiles of a share
    int steps;              // of a tile: R[0] R[1] R[2] / 4
    int KW;                 // waves that share the steps of a set's columns
    int G;                  // column groups
    int Mpad, Npad;
    int JG, planes, total, run;     // map groups, tap groups; workgroups in all and per XCD
    FastDiv dX4, dRX, dRY, dHX, dHY, dGU, dIU, dTG, dKX, dGB;     // R[2] / 4, R[2], R[1], H[2], H[1], GS / 16, IS / 16, columns of a map, k[2], GB
};

using GradFn = void (*)(GradTile);

// Bound by the matrix cores; next to them the copies of the tiles out of the caches.
template <int NJ, int NT>
__global__ void __launch_bounds__(64 * kGradWaves) k_wgrad_split(GradTile P)
{
    // two objects, so that the compiler knows that copies into one do not touch what is read from the other
    __shared__ __attribute__((aligned(16))) char bufA[kGradBuffer];
    __shared__ __attribute__((aligned(16))) char bufB[kGradBuffer];
    if (P.tiles < 0) {      // never taken: tells the optimizer that the buffers hold data
        reinterpret_cast<uintx4*>(bufA)[threadIdx.x] = P.gs[threadIdx.x];
        reinterpret_cast<uintx4*>(bufB)[threadIdx.x] = P.is[threadIdx.x];
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, grp = lane >> 4;
    const int set = wave / P.KW, kw = wave - set * P.KW, NG = kGradWaves / P.KW;
    // Workgroups go to the eight XCDs in turn; each takes a contiguous run, the groups of a share next to each other: they
    // read the same tiles.
    int id = (blockIdx.x & 7) * P.run + (blockIdx.x >> 3);
    if (id >= P.total) return;
    const int jg = id % P.JG; id /= P.JG;
    const int cg = id % P.G; id /= P.G;
    const int plane = id % P.planes, share = id / P.planes;
    const int ga = plane / P.planes_b, gb = plane - ga * P.planes_b;
    const int a0 = ga * P.GA, b0 = gb * P.GB;
    const int na = min(P.GA, P.k[0] - a0), nb = min(P.GB, P.k[1] - b0);
    const int tg = P.GA * P.GB * P.k[2];            // columns of an input map
    const int ncols = P.f * tg;
    const int n0 = cg * NT * NG * 16;
    const int i0 = n0 / tg, i1 = min(P.f - 1, (min(n0 + NT * NG * 16, ncols) - 1) / tg);
    const int nmaps = i1 - i0 + 1, mreal = min(NJ * 16, P.fo - jg * NJ * 16);
    const int itoff = NJ * 16 * P.GS;
    const int X4 = P.R[2] / 4;

    // the halo box starts at the shift of the group's last plane and row of taps
    const int sz = P.k[0] - a0 - na, sy = P.k[1] - b0 - nb;

    lds_bytes const lA = (lds_bytes)bufA, lB = (lds_bytes)bufB;
    int aoff[NJ], boff[NT];
#pragma unroll
    for (int jt = 0; jt < NJ; ++jt) aoff[jt] = (jt * 16 + col) * P.GS + grp * kVectorBytes;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int n = n0 + (set * NT + nt) * 16 + col;
        int o = 0;
        if (n < ncols) {
            const int i = (int)fdiv((unsigned)n, P.dTG), r = n - i * tg, q = (int)fdiv((unsigned)r, P.dKX), c = r - q * P.k[2];
            const int qa = (int)fdiv((unsigned)q, P.dGB), b = min(q - qa * P.GB, nb - 1), a = min(qa, na - 1);
            o = (i - i0) * P.IS + (((na - 1 - a) * P.H[1] + nb - 1 - b) * P.H[2] + P.k[2] - 1 - c) * kVectorBytes;
        }
        boff[nt] = itoff + o + grp * kVectorBytes;
    }
    // column tiles of this set that hold columns
    const int live = max(0, min(NT, ((min(n0 + NT * NG * 16, ncols) - n0 + 15) >> 4) - set * NT));

    // A wave's copies: span wave + 8 q of each of the two regions; lane's source within the tile, in 16-byte units, ~0: none.
    const int gu = P.GS / 16, iu = P.IS / 16;                   // units of a map in LDS
    const int span_g = (mreal * gu + 63) >> 6, span_i = (nmaps * iu + 63) >> 6;
    const int gbox = P.R[0] * P.R[1] * P.R[2] * 3, ibox = P.H[0] * P.H[1] * P.H[2] * 3;
    unsigned from[kGradSpans];
#pragma unroll
    for (int q = 0; q < kGradSpans; ++q) {
        const int sp = wave + q * kGradWaves;
        from[q] = ~0u;
        if (sp < span_g) {
            const int u = sp * 64 + lane, m = (int)fdiv((unsigned)u, P.dGU), e = u - m * gu, v = e / 3, part = e - v * 3;
            const int r = (int)fdiv((unsigned)v, P.dRX), x = v - r * P.R[2], z = (int)fdiv((unsigned)r, P.dRY), y = r - z * P.R[1];
            if (m < mreal && e < gbox) from[q] = ((((unsigned)m * P.P[0] + z) * P.P[1] + y) * P.P[2] + x) * 3 + part;
        } else if (sp - span_g < span_i) {
            const int u = (sp - span_g) * 64 + lane, m = (int)fdiv((unsigned)u, P.dIU), e = u - m * iu, v = e / 3, part = e - v * 3;
            const int r = (int)fdiv((unsigned)v, P.dHX), x = v - r * P.H[2], z = (int)fdiv((unsigned)r, P.dHY), y = r - z * P.H[1];
            if (m < nmaps && e < ibox) from[q] = ((((unsigned)m * P.I[0] + z) * P.I[1] + y) * P.I[2] + x) * 3 + part;
        }
    }
    const uintx4* const gsrc = P.gs + (long)jg * NJ * 16 * P.P[0] * P.P[1] * P.P[2] * 3;
    const uintx4* const isrc = P.is + (((long)i0 * P.I[0] + sz) * P.I[1] + sy) * P.I[2] * 3;
    // The next tile to be copied, stepped without divisions: vectors (g: in gs, i: in is) in front of it on every axis and its
    // number within the residue.  The pieces of a residue are k - 1 vectors longer in `is`.
    const int first = share * P.tps, last = min(first + P.tps, P.tiles);
    int gx, ix, qx, gy, iy, qy, gz, iz, qz;
    {
        const int r = first / P.tiles_x, tx = first - r * P.tiles_x, tz = r / P.tiles_y, ty = r - tz * P.tiles_y;
        const int hx = tx / P.T[2], hy = ty / P.T[1], hz = tz / P.T[0];
        qx = tx - hx * P.T[2]; qy = ty - hy * P.T[1]; qz = tz - hz * P.T[0];
        gx = tx * P.R[2]; gy = ty * P.R[1]; gz = tz * P.R[0];
        ix = gx + hx * (P.k[2] - 1); iy = gy + hy * (P.k[1] - 1); iz = gz + hz * (P.k[0] - 1);
    }
    auto copy_tile = [&](char* buf, int& odd) __attribute__((always_inline)) {
        odd = gx / 4 + gy + gz;         // sign of its first step
        const uintx4* g = gsrc + (((long)gz * P.P[1] + gy) * P.P[2] + gx) * 3;
        const uintx4* in = isrc + (((long)iz * P.I[1] + iy) * P.I[2] + ix) * 3;
#pragma unroll
        for (int q = 0; q < kGradSpans; ++q) {
            const int sp = wave + q * kGradWaves;
            if (sp >= span_g + span_i) break;                                           // uniform
            const bool i = sp >= span_g;                                                // uniform
            char* at = i ? buf + itoff + (sp - span_g) * 1024 : buf + sp * 1024;        // uniform
            const uintx4* base = i ? in : g;                                            // uniform
            unsigned f = from[q];
            asm volatile("" : "+v"(f));     // the 64-bit address is made here, and not kept in registers from tile to tile
            if (f != ~0u) __builtin_amdgcn_global_load_lds((global_cptr)(base + f), (lds_ptr)at, 16, 0, 0);
        }
        gx += P.R[2]; ix += P.R[2];
        if (++qx == P.T[2]) { qx = 0; ix += P.k[2] - 1; }
        if (gx < P.P[2]) return;
        gx = ix = 0; gy += P.R[1]; iy += P.R[1];
        if (++qy == P.T[1]) { qy = 0; iy += P.k[1] - 1; }
        if (gy < P.P[1]) return;
        gy = iy = 0; gz += P.R[0]; iz += P.R[0];
        if (++qz == P.T[0]) { qz = 0; iz += P.k[0] - 1; }
    };

    floatx4 acc[NJ][NT];
#pragma unroll
    for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[jt][nt] = floatx4{0.f, 0.f, 0.f, 0.f};

    // rows of maps that do not exist stay zero
    for (int q = mreal * gu + threadIdx.x; q < NJ * 16 * gu; q += 64 * kGradWaves) {
        reinterpret_cast<uintx4*>(bufA)[q] = uintx4{0u, 0u, 0u, 0u};
        reinterpret_cast<uintx4*>(bufB)[q] = uintx4{0u, 0u, 0u, 0u};
    }
    __syncthreads();

    // The wave's steps of a staged tile.  The copies of the next tile are queued behind the requests for the first operands.
    auto use_tile = [&](lds_bytes buf, int odd, bool more, char* other, int& other_odd) __attribute__((always_inline)) {
        auto load = [&](uintx4 (&v)[3], lds_bytes at) {
#pragma unroll
            for (int p = 0; p < 3; ++p) v[p] = reinterpret_cast<lds_quads>(at)[p];
        };
        int ks = kw;
        if (live == 0 || ks >= P.steps) {       // uniform
            if (more) copy_tile(other, other_odd);
            return;
        }
        for (; ks < P.steps; ks += P.KW) {
            const int r = (int)fdiv((unsigned)ks, P.dX4), x = (ks - r * X4) * 4, z = (int)fdiv((unsigned)r, P.dRY), y = r - z * P.R[1];
            const int ao = (r * P.R[2] + x) * kVectorBytes, bo = ((z * P.H[1] + y) * P.H[2] + x) * kVectorBytes;
            const float sign = (odd + x / 4 + y + z) & 1 ? -kUnscale : kUnscale;
            bf16x8 a[NJ][3];
            uintx4 b0[3], b1[3];
            floatx4 t0[NJ], t1[NJ];
            load(b0, buf + boff[0] + bo);
#pragma unroll
            for (int q = 0; q < 3; ++q)     // in the order the products need them
#pragma unroll
                for (int jt = 0; jt < NJ; ++jt) {
                    const int p = q == 0 ? 0 : 3 - q;
                    a[jt][p] = __builtin_bit_cast(bf16x8, reinterpret_cast<lds_quads>(buf + aoff[jt] + ao)[p]);
                }
            __builtin_amdgcn_sched_barrier(0);
            if (more && ks == kw) copy_tile(other, other_odd);
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) t1[jt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                uintx4 (&b)[3] = nt & 1 ? b1 : b0;
                uintx4 (&bn)[3] = nt & 1 ? b0 : b1;
                const lds_bytes at = buf + boff[nt + 1 < NT ? nt + 1 : 0] + bo;
                auto request = [&](int slot) __attribute__((always_inline)) {
                    const int p = (slot + 2) % 3;       // in the order that the products need them
                    if (nt + 1 < NT && slot < 3) bn[p] = reinterpret_cast<lds_quads>(at)[p];
                };
                floatx4 *into[NJ];
#pragma unroll
                for (int jt = 0; jt < NJ; ++jt) into[jt] = &acc[jt][nt ? nt - 1 : 0];
                products<NJ, 0, (NJ > 1)>(nt & 1 ? t1 : t0, a, b, nt & 1 ? t0 : t1, sign, into, request);
            }
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) add_signed<0>(acc[jt][NT - 1], (NT - 1) & 1 ? t1[jt] : t0[jt], sign);
        }
    };

    int oddA = 0, oddB = 0;
    if (first < last) copy_tile(bufA, oddA);
    for (int tile = first; tile < last; tile += 2) {
        __builtin_amdgcn_s_waitcnt(0);      // this wave's copies have landed
        __syncthreads();                    // everyone's have, and nobody still reads the other buffer
        use_tile(lA, oddA, tile + 1 < last, bufB, oddB);
        if (tile + 1 >= last) break;
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        use_tile(lB, oddB, tile + 2 < last, bufA, oddA);
    }

    // Sums that are not finite: the parts of an infinity or a NaN do not multiply as it does.  Where the first products of the wave's
    // share, in fp32, make NaN of all of them already -- whole maps of a net that has diverged -- NaN they are, and the finite ones
    // stand; else its share again in fp32, straight from memory.  40 -> 40 maps, 64^3, 5^3, 585 us on finite values: all NaN 600 us,
    // one voxel or all of them infinite 2400 us.
    bool bad = false;
#pragma unroll
    for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int r = 0; r < 4; ++r) bad = bad || !(fabsf(acc[jt][nt][r]) <= kLargest);
    if (__builtin_amdgcn_ballot_w64(bad)) {
        // the launch's parameters from memory again: they need not stay in scalar registers for this
        auto args = __builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(args));
        const GradTile& C = *(const GradTile*)args;
        const int tg = C.GA * C.GB * C.k[2], ncols = C.f * tg, X4 = C.R[2] / 4;
        const long ovol = (long)C.o[0] * C.o[1] * C.o[2], nvol = (long)C.n[0] * C.n[1] * C.n[2];
        // voxel of the lane in step ks of a tile, piece e; false: none
        auto voxel = [&](int tile, int ks, int e, int& z, int& y, int& x) {
            const int tx = tile % C.tiles_x, tr = tile / C.tiles_x, ty = tr % C.tiles_y, tz = tr / C.tiles_y;
            const int r = ks / X4, qx = tx % C.T[2] * C.R[2] + (ks - r * X4) * 4 + grp;
            const int qy = C.q0[1] + ty % C.T[1] * C.R[1] + r % C.R[1], qz = C.q0[0] + tz % C.T[0] * C.R[0] + r / C.R[1];
            const int ex = e % C.E[2], ey = e / C.E[2] % C.E[1], ez = e / C.E[2] / C.E[1];
            z = C.r0[0] + tz / C.T[0] + (ez * C.Q[0] + qz) * C.sp[0];
            y = C.r0[1] + ty / C.T[1] + (ey * C.Q[1] + qy) * C.sp[1];
            x = tx / C.T[2] + (ex * C.Q[2] + qx) * C.sp[2];
            return qz < C.Q[0] && qy < C.Q[1] && qx < C.Q[2] && z < C.o[0] && y < C.o[1] && x < C.o[2];
        };
        auto of_gout = [&](int jt, bool ok, int z, int y, int x) {
            const int j = (jg * NJ + jt) * 16 + col;
            return ok && j < C.fo ? ((global_floats)C.gout)[j * ovol + ((long)z * C.o[1] + y) * C.o[2] + x] : 0.f;
        };
        // where the lane's column of a tile begins in `in`, -1: none
        auto column = [&](int nt) {
            const int n = n0 + (set * NT + nt) * 16 + col;
            const int i = n / tg, q = n - i * tg, c = q % C.k[2], b = b0 + q / C.k[2] % C.GB, a = a0 + q / C.k[2] / C.GB;
            const int cz = C.sp[0] * (C.k[0] - 1 - a), cy = C.sp[1] * (C.k[1] - 1 - b), cx = C.sp[2] * (C.k[2] - 1 - c);
            return n < ncols && a < C.k[0] && b < C.k[1] ? i * nvol + ((long)cz * C.n[1] + cy) * C.n[2] + cx : -1l;
        };
        auto of_in = [&](long begin, bool ok, int z, int y, int x) {
            return ok && begin >= 0 ? ((global_floats)C.in)[begin + ((long)z * C.n[1] + y) * C.n[2] + x] : 0.f;
        };
        auto is_wrong = [](float v) {
            asm volatile("" : "+v"(v));     // compared anew: outcomes that are kept would take all scalar registers
            return !(fabsf(v) <= kLargest);
        };
        bool open = false;          // whether some sums are not NaN after these products (uniform)
#pragma unroll 1
        for (int p = 0; p < NT && !open; ++p) {
            unsigned wrong = 0;     // the lane's sums in column tile p that are, where they are wanted
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                if (p == nt) {      // uniform
#pragma unroll
                    for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (is_wrong(acc[jt][nt][r])) wrong |= 1u << (jt * 4 + r);
                }
            const long begin = column(p);
            if (begin < 0) wrong = 0;
            floatx4 t[NJ];
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt) t[jt] = floatx4{0.f, 0.f, 0.f, 0.f};
            for (int e = 0; e < 8; ++e) {
                int z, y, x;
                const bool ok = voxel(first, kw, e, z, y, x) && kw < C.steps;
                const float bv = of_in(begin, ok, z, y, x);
#pragma unroll
                for (int jt = 0; jt < NJ; ++jt) t[jt] = __builtin_amdgcn_mfma_f32_16x16x4f32(of_gout(jt, ok, z, y, x), bv, t[jt], 0, 0, 0);
            }
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (t[jt][r] != t[jt][r]) wrong &= ~(1u << (jt * 4 + r));
            open = __builtin_amdgcn_ballot_w64(wrong != 0) != 0;
        }
        if (!open) {
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[jt][nt][r] = is_wrong(acc[jt][nt][r]) ? __builtin_nanf("") : acc[jt][nt][r];
        } else {
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[jt][nt] = floatx4{0.f, 0.f, 0.f, 0.f};
            long begin[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) begin[nt] = column(nt);
            for (int tile = first; tile < last; ++tile)
                for (int ks = kw; ks < C.steps; ks += C.KW)
                    for (int e = 0; e < 8; ++e) {
                        int z, y, x;
                        const bool ok = voxel(tile, ks, e, z, y, x);
                        float av[NJ], bv[NT];
#pragma unroll
                        for (int jt = 0; jt < NJ; ++jt) av[jt] = of_gout(jt, ok, z, y, x);
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) bv[nt] = of_in(begin[nt], ok, z, y, x);
#pragma unroll
                        for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
                            for (int nt = 0; nt < NT; ++nt)
                                acc[jt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[jt], bv[nt], acc[jt][nt], 0, 0, 0);
                    }
        }
    }

    // add the sums of the KW waves of each set, pairs first
    auto slot = [&](int q) { return reinterpret_cast<floatx4*>(q < 2 ? bufA : bufB) + (q & 1) * (NJ * NT * 64) + lane; };   // four at most
    for (int h = P.KW / 2; h >= 1; h /= 2) {
        __syncthreads();
        if (kw >= h && kw < 2 * h) {
            floatx4* to = slot(set * h + kw - h);
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) to[(jt * NT + nt) * 64] = acc[jt][nt];
        }
        __syncthreads();
        if (kw < h) {
            const floatx4* of = slot(set * h + kw);
#pragma unroll
            for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[jt][nt] += of[(jt * NT + nt) * 64];
        }
    }
    if (kw == 0 && live > 0) {
        float* out = P.partial + ((long)(share * P.planes + plane) * P.Mpad + jg * NJ * 16) * P.Npad + (cg * NG + set) * NT * 16;
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (nt < live && jt * 16 + grp * 4 + r < mreal) {
                        float* at = out + (long)(jt * 16 + grp * 4 + r) * P.Npad + nt * 16 + col;
                        *at = P.more ? *at + acc[jt][nt][r] : acc[jt][nt][r];
                    }
    }
}

}  // namespace split
}  // namespace znn
