// FFT method on overlapping tiles (overlap-save / overlap-add).
//
// The transform of a whole volume needs one product per edge and frequency of the VOLUME; cut into tiles of
// M voxels per axis that advance by B = M - S + 1 (S = s (k - 1) + 1: span of the kernel), a layer needs one
// product per edge, tile and frequency of a TILE instead.  The number of products grows by (M / B)^3, but
// the kernel spectra shrink by the ratio of the volumes (96^3 images, 7^3 kernels, M = 24: 0.86 GB instead of 52 GB,
// or of 3.8 GB transformed along two axes), the tile index becomes a matrix dimension -- the multiply-accumulate of
// a frequency is a matrix product [f'][f] x [f][tiles], that of the kernel gradient [f'][tiles] x [tiles][f] --
// and matrix products run on the matrix cores, with every spectrum element read once per pass instead of once
// per result node.  A tile's 3D transform fits one workgroup's LDS, so it is one trip through memory.
//
//   forward   out on [t B, t B + B) = crop_{[S-1, M)} IFFT( sum_i W^[j][i] U^[i][t] ),   U = in on [t B, t B + M)
//   backward  gin += at t B           IFFT( sum_j conj(W^[j][i]) V^[j][t] ),             V = gout on [t B, t B + B) from S - 1 on
//   gradient  gw  = lags s a of       IFFT( sum_t V^[j][t] conj(U^[i][t]) )
// (derivation: circular products of length M are free of wrap-around because B + S - 1 = M).
//
// Spectra are stored in blocks of 16 frequencies, [frequency block][map][tile][16]: a tile's transform stores full
// 128-byte lines, and the matrix product of a block reads its operands as runs of 128 bytes.
#include "fft_reg_impl.h"
#include "fft_tile.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace znn {

namespace {

constexpr int kTileThreads = 512;           // most threads of a transform workgroup
constexpr int kTileEntries = 16;            // most tiles of a transform workgroup
constexpr size_t kTileLds = 60 * 1024;   // LDS of a transform workgroup: two fit a compute unit
constexpr size_t kUnitLds = 160 * 1024, kTileStatic = 512;      // LDS of a compute unit; of a workgroup beside its tiles

// ---------------------------------------------------------------- transforms of tiles
// An entry is one tile of one map (for kernels: one kernel).  Axis order z, y, x everywhere.
struct TileGeom {
    int M[3], Mxh;              // transform lengths, M[2] / 2 + 1
    int T[3], hop[3];           // tiles per axis, voxels from one tile to the next
    int n[3];                   // extents of the real maps
    int w[3];                   // samples a tile holds per axis: element o + i * sp of the transform, i < w
    int o[3], sp[3];
    unsigned mask[3];           // bit m: element m holds a sample
    int entries, per_wg;        // entries in all, entries per workgroup
    int vw, clip;               // samples per memory access along x: 4, 2 or 1; tiles reach beyond the map
    int rows_per_step, step[3]; // rows a workgroup's threads cover at a time, and that as (entries, z, y)
    FastDiv fw[3], fwx, fMxh, fcol;     // divisions by w, w[2] / vw, Mxh, My * Mxh
    int first, count;           // tiles of a map in this launch: numbers first .. first + count - 1 (finish_geom: 0 = all)
};
struct TileFwd { const float* src; float2* dst; TileGeom G; };
struct TileInv { const float2* src; float* dst; TileGeom G; float scale; int splits; long split_stride; Finish finish; };

struct EntryInfo { long base; int v[3]; int map; };

// where an entry's samples lie in the real maps, and how many of them per axis exist
__device__ __forceinline__ EntryInfo entry_info(const TileGeom& G, int e)
{
    EntryInfo I;
    if (e >= G.entries) { I.base = 0; I.v[0] = I.v[1] = I.v[2] = I.map = 0; return I; }
    const int map = I.map = e / G.count;
    int t = G.first + e - map * G.count;
    const int tz = t / (G.T[1] * G.T[2]);
    t -= tz * G.T[1] * G.T[2];
    const int ty = t / G.T[2], tx = t - ty * G.T[2];
    const int z0 = tz * G.hop[0], y0 = ty * G.hop[1], x0 = tx * G.hop[2];
    I.base = (((long)map * G.n[0] + z0) * G.n[1] + y0) * (long)G.n[2] + x0;
    I.v[0] = min(G.w[0], G.n[0] - z0);
    I.v[1] = min(G.w[1], G.n[1] - y0);
    I.v[2] = min(G.w[2], G.n[2] - x0);
    return I;
}

// Lengths 2^a q with q = 3 or 5 are taken apart by the prime factor algorithm: element q n1 + 2^a n2 (mod M) goes to place n1 of
// transform n2, and coefficient (k1, k2) is that of the k with these residues, so nothing is multiplied by twiddles in between, and all
// indices are of registers (24 points: 264 instead of 320 operations).
constexpr int odd_part(int n) { return n % 2 ? n : odd_part(n / 2); }

template <int M, int DIR>
__device__ __forceinline__ void fft_inplace(float2 (&v)[M])
{
    constexpr int Q = odd_part(M), P = M / Q;
    if constexpr (Q > 1 && P > 1) {
        float2 t[Q][P];
#pragma unroll
        for (int n2 = 0; n2 < Q; ++n2) {
#pragma unroll
            for (int n1 = 0; n1 < P; ++n1) t[n2][n1] = v[(Q * n1 + P * n2) % M];
            fft_inplace<P, DIR>(t[n2]);
        }
#pragma unroll
        for (int k1 = 0; k1 < P; ++k1) {
            float2 c[Q];
#pragma unroll
            for (int n2 = 0; n2 < Q; ++n2) c[n2] = t[n2][k1];
            fft_inplace<Q, DIR>(c);
#pragma unroll
            for (int j = 0; j < Q; ++j) v[k1 + P * j] = c[(k1 + P * j) % Q];
        }
    } else if constexpr (M > 1) {
        float2 w[M];
        passes<M, DIR, M, 1>(v, w);
        if constexpr (count_passes(M) % 2 == 1) {
#pragma unroll
            for (int m = 0; m < M; ++m) v[m] = w[m];
        }
    }
}

// real row of M samples at `row` (masked) -> M/2 + 1 coefficients in the same words, by one thread.  With a = Z[k], b = Z[H - k],
// e = a + conj b and u = -i w^k (a - conj b): X[k] = (e + u) / 2 and X[H - k] = conj(e - u) / 2.
template <int M, bool FULL>
__device__ __forceinline__ void row_r2c(float2* row, unsigned mask)
{
    constexpr int H = M / 2;
    static_assert(H % 2 == 0, "");
    float2 Z[H];
#pragma unroll
    for (int m = 0; m < H; ++m) {
        const float2 v = row[m];
        Z[m].x = FULL || ((mask >> (2 * m)) & 1u) ? v.x : 0.f;
        Z[m].y = FULL || ((mask >> (2 * m + 1)) & 1u) ? v.y : 0.f;
    }
    fft_inplace<H, -1>(Z);
    row[0] = make_float2(Z[0].x + Z[0].y, 0.f);
    row[H] = make_float2(Z[0].x - Z[0].y, 0.f);
    row[H / 2] = make_float2(Z[H / 2].x, -Z[H / 2].y);
#pragma unroll
    for (int k = 1; k < H / 2; ++k) {
        const float2 a = Z[k], b = Z[H - k];
        const float ex = 0.5f * (a.x + b.x), ey = 0.5f * (a.y - b.y), dx = a.x - b.x, dy = a.y + b.y;
        const float wc = 0.5f * TwTable<M>::t.c[k], ws = -0.5f * TwTable<M>::t.s[k];
        const float ux = wc * dy + ws * dx, uy = ws * dy - wc * dx;
        row[k] = make_float2(ex + ux, ey + uy);
        row[H - k] = make_float2(ex - ux, uy - ey);
    }
}

// M/2 + 1 coefficients -> M real samples (times M) in the same words.  Z[k] = e + u and Z[H - k] = conj(e - u) with a = X[k], b = X[H - k],
// e = a + conj b and u = i w^-k (a - conj b).
template <int M>
__device__ __forceinline__ void row_c2r(float2* row)
{
    constexpr int H = M / 2;
    static_assert(H % 2 == 0, "");
    float2 X[H + 1], Z[H];
#pragma unroll
    for (int k = 0; k <= H; ++k) X[k] = row[k];
    Z[0] = make_float2(X[0].x + X[H].x, X[0].x - X[H].x);
    Z[H / 2] = make_float2(2.f * X[H / 2].x, -2.f * X[H / 2].y);
#pragma unroll
    for (int k = 1; k < H / 2; ++k) {
        const float2 a = X[k], b = X[H - k];
        const float ex = a.x + b.x, ey = a.y - b.y, dx = a.x - b.x, dy = a.y + b.y;
        const float wc = TwTable<M>::t.c[k], ws = TwTable<M>::t.s[k];          // w^-k
        const float ux = -wc * dy - ws * dx, uy = wc * dx - ws * dy;
        Z[k] = make_float2(ex + ux, ey + uy);
        Z[H - k] = make_float2(ex - ux, uy - ey);
    }
    fft_inplace<H, +1>(Z);
#pragma unroll
    for (int m = 0; m < H; ++m) row[m] = Z[m];
}

template <int M, bool FULL>
__device__ __forceinline__ void rows_r2c(float2* lds, const TileGeom& G)
{
    const int rows = G.per_wg * G.w[0] * G.w[1];
    for (int u = threadIdx.x; u < rows; u += blockDim.x) {
        const int q = (int)fdiv((unsigned)u, G.fw[1]), y = u - q * G.w[1];
        const int b = (int)fdiv((unsigned)q, G.fw[0]), z = q - b * G.w[0];
        row_r2c<M, FULL>(lds + ((b * G.w[0] + z) * G.M[1] + G.o[1] + y * G.sp[1]) * G.Mxh, G.mask[2]);
    }
}

template <int M>
__device__ __forceinline__ void rows_c2r(float2* lds, const TileGeom& G)
{
    const int rows = G.per_wg * G.w[0] * G.w[1];
    for (int u = threadIdx.x; u < rows; u += blockDim.x) {
        const int q = (int)fdiv((unsigned)u, G.fw[1]), y = u - q * G.w[1];
        const int b = (int)fdiv((unsigned)q, G.fw[0]), z = q - b * G.w[0];
        row_c2r<M>(lds + ((b * G.w[0] + z) * G.M[1] + G.o[1] + y * G.sp[1]) * G.Mxh);
    }
}

// The mask of an axis as the loops test it, bit by bit: without this the compiler keeps every bit's test in scalar registers
// from one column to the next, three times as many as there are.
__device__ __forceinline__ unsigned bits(unsigned mask)
{
    asm volatile("" : "+s"(mask));
    return mask;
}

// transforms along y, in place, of the planes z that hold samples; forward reads, inverse writes only the
// rows of mask[1]
template <int M, int DIR, bool FULL>
__device__ __forceinline__ void columns_y(float2* lds, const TileGeom& G)
{
    const int cols = G.per_wg * G.w[0] * G.Mxh;
    for (int u = threadIdx.x; u < cols; u += blockDim.x) {
        const int q = (int)fdiv((unsigned)u, G.fMxh), k = u - q * G.Mxh;
        const int b = (int)fdiv((unsigned)q, G.fw[0]), z = q - b * G.w[0];
        float2* c = lds + (b * G.w[0] + z) * G.M[1] * G.Mxh + k;
        const unsigned mask = bits(G.mask[1]);
        float2 v[M];
#pragma unroll
        for (int m = 0; m < M; ++m)
            v[m] = FULL || ((mask >> m) & 1u) ? c[m * G.Mxh] : make_float2(0.f, 0.f);
        fft_inplace<M, DIR>(v);
        // stepped anew: the places of all elements would take the registers of a workgroup's share of the unit
        int at = (int)(c - lds);
        asm volatile("" : "+v"(at));
#pragma unroll
        for (int m = 0; m < M; ++m, at += G.Mxh)
            if (DIR < 0 || ((mask >> m) & 1u)) lds[at] = v[m];
    }
}

// Frequency w = m P + p of an entry lies at block w / 16, element w % 16.  (m P) mod 16 takes four values (P = My Mxh is
// a multiple of 4), so a thread keeps four byte offsets and the rest is uniform: block (m P) / 16 is a scalar address.
struct BlockOffsets {
    unsigned at[4];
    __device__ __forceinline__ BlockOffsets(int p, int P, unsigned blk_bytes)
    {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int t = p + ((r * P) & 15);
            at[r] = (unsigned)(t >> 4) * blk_bytes + (unsigned)(t & 15) * 8u;
        }
    }
};

// forward transforms along z and the store of the spectra
template <int M, bool FULL>
__device__ __forceinline__ void columns_z_store(const float2* lds, float2* dst, const TileGeom& G, int e0)
{
    const int P = G.M[1] * G.Mxh;
    const int cols = G.per_wg * P;
    const unsigned blk = (unsigned)G.entries * 128u;
    for (int u = threadIdx.x; u < cols; u += blockDim.x) {
        const int b = (int)fdiv((unsigned)u, G.fcol), p = u - b * P;
        if (e0 + b >= G.entries) break;
        const float2* c = lds + b * G.w[0] * P + p;
        const unsigned mask = bits(G.mask[0]);
        float2 v[M];
#pragma unroll
        for (int m = 0; m < M; ++m) {
            v[m] = make_float2(0.f, 0.f);
            if (FULL || ((mask >> m) & 1u)) { v[m] = *c; c += P; }
        }
        fft_inplace<M, -1>(v);
        char* d = reinterpret_cast<char*>(dst + (long)e0 * 16);
        const BlockOffsets off(p, P, blk);
#pragma unroll
        for (int m = 0; m < M; ++m)
            *reinterpret_cast<float2*>(d + (long)((m * P) >> 4) * blk + (off.at[m & 3] + (unsigned)b * 128u)) = v[m];
    }
}

// load of the spectra (splits: partial sums to be added, in ascending order) and inverse transforms along z
template <int M, bool SPLIT>
__device__ __forceinline__ void load_columns_z(float2* lds, const TileInv& I, int e0)
{
    const TileGeom& G = I.G;
    const int P = G.M[1] * G.Mxh;
    const int cols = G.per_wg * P;
    const unsigned blk = (unsigned)G.entries * 128u;
    for (int u = threadIdx.x; u < cols; u += blockDim.x) {
        const int b = (int)fdiv((unsigned)u, G.fcol), p = u - b * P;
        if (e0 + b >= G.entries) break;
        const char* s = reinterpret_cast<const char*>(I.src + (long)e0 * 16);
        const BlockOffsets off(p, P, blk);
        float2 v[M];
#pragma unroll
        for (int m = 0; m < M; ++m)
            v[m] = *reinterpret_cast<const float2*>(s + (long)((m * P) >> 4) * blk + (off.at[m & 3] + (unsigned)b * 128u));
        for (int r = 1; SPLIT && r < I.splits; ++r) {
            s += I.split_stride * 8;
#pragma unroll
            for (int m = 0; m < M; ++m)
                v[m] = cadd(v[m], *reinterpret_cast<const float2*>(s + (long)((m * P) >> 4) * blk + (off.at[m & 3] + (unsigned)b * 128u)));
        }
        fft_inplace<M, +1>(v);
        float2* c = lds + b * G.w[0] * P + p;
        const unsigned mask = bits(G.mask[0]);
#pragma unroll
        for (int m = 0; m < M; ++m)
            if ((mask >> m) & 1u) { *c = v[m]; c += P; }
    }
}

// 2D layers have no z transform: the spectra go from or to LDS as they are
__device__ __forceinline__ void store_plane(const float2* lds, float2* dst, const TileGeom& G, int e0)
{
    const int P = G.M[1] * G.Mxh, total = min(G.per_wg, G.entries - e0) * P;
#pragma unroll 8
    for (int u = threadIdx.x; u < total; u += blockDim.x) {
        const int b = (int)fdiv((unsigned)u, G.fcol), p = u - b * P;
        dst[((long)(p >> 4) * G.entries + e0 + b) * 16 + (p & 15)] = lds[u];
    }
}

__device__ __forceinline__ void load_plane(float2* lds, const TileInv& I, int e0)
{
    constexpr int kLoads = 8;
    const TileGeom& G = I.G;
    const int P = G.M[1] * G.Mxh, total = min(G.per_wg, G.entries - e0) * P;
    for (int u0 = threadIdx.x; u0 < total; u0 += kLoads * blockDim.x) {
        float2 v[kLoads];
        const float2* s = I.src;
        for (int r = 0; r < I.splits; ++r, s += I.split_stride) {
            float2 t[kLoads];
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                const int u = min(u0 + i * (int)blockDim.x, total - 1);
                const int b = (int)fdiv((unsigned)u, G.fcol), p = u - b * P;
                t[i] = s[((long)(p >> 4) * G.entries + e0 + b) * 16 + (p & 15)];
            }
#pragma unroll
            for (int i = 0; i < kLoads; ++i) v[i] = r ? cadd(v[i], t[i]) : t[i];
        }
#pragma unroll
        for (int i = 0; i < kLoads; ++i)
            if (u0 + i * (int)blockDim.x < total) lds[u0 + i * blockDim.x] = v[i];
    }
}

// The samples of the workgroup's entries travel VW at a time (VW divides the window along x), kBatch accesses per thread
// in flight: a workgroup waits for memory once or twice, not once per few rows.
constexpr int kBatch = 12;
typedef float floatu4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float floatu2 __attribute__((ext_vector_type(2), aligned(4)));
template <int VW> struct VecOf;
template <> struct VecOf<4> { typedef floatu4 type; };
template <> struct VecOf<2> { typedef floatu2 type; };
template <> struct VecOf<1> { typedef float type; };

// A thread's x position stays fixed; its rows are `rows_per_step` apart, and (entry, z, y) are stepped in mixed radix
// without divisions (32-bit multiplications by constants of the launch would run at a quarter of the rate).
struct RowWalk {
    int x, b, z, y;
    bool idle;
    __device__ __forceinline__ RowWalk(const TileGeom& G, int vw)
    {
        const int t = threadIdx.x, r = (int)fdiv((unsigned)t, G.fwx);
        x = (t - r * (G.w[2] / vw)) * vw;
        const int q = (int)fdiv((unsigned)r, G.fw[1]);
        y = r - q * G.w[1];
        b = (int)fdiv((unsigned)q, G.fw[0]);
        z = q - b * G.w[0];
        idle = r >= G.rows_per_step;
    }
    __device__ __forceinline__ void step(const TileGeom& G)
    {
        y += G.step[2];
        const int cy = y >= G.w[1] ? 1 : 0;
        y -= cy ? G.w[1] : 0;
        z += G.step[1] + cy;
        const int cz = z >= G.w[0] ? 1 : 0;
        z -= cz ? G.w[0] : 0;
        b += G.step[0] + cz;
    }
    __device__ __forceinline__ int lds_at(const TileGeom& G) const
    {
        const int row = (int)__umul24(__umul24(b, G.w[0]) + z, G.M[1]) + G.o[1] + (int)__umul24(y, G.sp[1]);
        return (int)__umul24(row, 2 * G.Mxh) + G.o[2] + x * G.sp[2];
    }
    // samples of the row from x on that exist
    __device__ __forceinline__ int left(const EntryInfo& E) const { return y < E.v[1] && z < E.v[0] ? E.v[2] - x : 0; }
    __device__ __forceinline__ long at(const TileGeom& G, const EntryInfo& E) const
    {
        return E.base + ((long)(z * G.n[1] + y) * G.n[2] + x);
    }
};

// All loads of a batch are unconditional (a branch around one makes the compiler wait for it before the next: 25 000
// clocks per tile instead of 2 500): coordinates outside the map are clamped into it and the values replaced by zeros.
// CLIP: some tiles of the launch reach beyond the map; a row that ends inside the vector is loaded from further left
// (every tile holds at least VW samples per row) and shifted.
template <int VW, bool CLIP>
__device__ __forceinline__ void load_samples(float* lf, const float* __restrict__ src, const TileGeom& G, const EntryInfo* info)
{
    typedef typename VecOf<VW>::type vec;
    RowWalk R(G, VW);
    if (R.idle) return;
    while (R.b < G.per_wg) {
        vec v[kBatch];
        int at[kBatch];                 // LDS word, and from bit 16 on the samples that exist; -1: no row left
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const EntryInfo& E = info[min(R.b, G.per_wg - 1)];
            at[i] = R.b < G.per_wg ? R.lds_at(G) : -1;
            if constexpr (CLIP) {
                const int left = min(VW, max(0, R.left(E)));
                if (R.b < G.per_wg) at[i] |= left << 16;
                const int z = max(0, min(R.z, E.v[0] - 1)), y = max(0, min(R.y, E.v[1] - 1));
                const int x = left > 0 ? R.x - (VW - left) : 0;
                v[i] = *reinterpret_cast<const vec*>(src + E.base + ((long)(z * G.n[1] + y) * G.n[2] + x));
            } else {
                v[i] = *reinterpret_cast<const vec*>(src + (R.b < G.per_wg ? R.at(G, E) : 0));
            }
            R.step(G);
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
            if (at[i] >= 0) {
                float t[VW];
                __builtin_memcpy(t, &v[i], sizeof(vec));
                if constexpr (CLIP) {
                    const int left = at[i] >> 16, d = VW - left;
                    if constexpr (VW >= 2) {
#pragma unroll
                        for (int bit = 1; bit < VW; bit *= 2)
#pragma unroll
                            for (int c = 0; c + bit < VW; ++c) {        // ascending: reads what is not yet shifted
                                float here = t[c], next = t[c + bit];
                                asm volatile("" : "+v"(here), "+v"(next));      // a choice between registers; else it becomes one of a place in scratch memory
                                t[c] = d & bit ? next : here;
                            }
                    }
#pragma unroll
                    for (int c = 0; c < VW; ++c) t[c] = c < left ? t[c] : 0.f;
                }
#pragma unroll
                for (int c = 0; c < VW; ++c) lf[(at[i] & 0xffff) + c * G.sp[2]] = t[c];
            }
    }
}

// What follows the sums of an image (Finish, the rectifier) is done as they are stored.  A pass of its own over the image took 17 us beside the 36
// of the transform on 40 maps of 23 x 75 x 125, and 4 us where there is little of it.
template <int VW, bool FINISH>
__device__ __forceinline__ void store_samples(const float* lf, const TileInv& A, const EntryInfo* info, const float* bias)
{
    const TileGeom& G = A.G;
    const Finish& F = A.finish;
    typedef typename VecOf<VW>::type vec;
    RowWalk R(G, VW);
    if (R.idle) return;
#pragma unroll 4
    while (R.b < G.per_wg) {
        const EntryInfo& E = info[R.b];
        const int at = R.lds_at(G), left = R.left(E);
        const long place = R.at(G, E);
        float* p = A.dst + place;
        float v[VW];
#pragma unroll
        for (int c = 0; c < VW; ++c) v[c] = A.scale * lf[at + c * G.sp[2]];
        if (FINISH && F.deriv) {                        // uniform, as F.y
#pragma unroll
            for (int c = 0; c < VW; ++c)
                if (c < left) v[c] = F.deriv[place + c] > 0.f ? v[c] : 0.f;
        }
        if (FINISH && F.y) {
#pragma clang fp contract(off)                          // of the sum that is stored
            float u[VW];
#pragma unroll
            for (int c = 0; c < VW; ++c) { u[c] = v[c] + bias[R.b]; u[c] = u[c] > 0.f ? u[c] : 0.f; }
            if (left >= VW) {
                vec t;
                __builtin_memcpy(&t, u, sizeof(vec));
                *reinterpret_cast<vec*>(F.y + place) = t;
            } else {
#pragma unroll
                for (int c = 0; c < VW; ++c)
                    if (c < left) F.y[place + c] = u[c];
            }
        }
        if (left >= VW) {
            vec t;
            __builtin_memcpy(&t, v, sizeof(vec));
            *reinterpret_cast<vec*>(p) = t;
        } else {
#pragma unroll
            for (int c = 0; c < VW; ++c)
                if (c < left) p[c] = v[c];
        }
        R.step(G);
    }
}

// one pass of a workgroup, by the transform length of its axis (LONG: the kernel instance that also takes length 32)
#define ZNN_TILE_SWITCH(LONG, L, CALL1, CALL)                             \
    switch (L) {                                                          \
        case 1: CALL1; break;                                             \
        case 8: CALL(8); break;                                           \
        case 12: CALL(12); break;                                         \
        case 16: CALL(16); break;                                         \
        case 20: CALL(20); break;                                         \
        case 24: CALL(24); break;                                         \
        default: if constexpr (LONG) CALL(32); break;                     \
    }

typedef __attribute__((address_space(1))) const void* global_cptr;
typedef __attribute__((address_space(3))) void* lds_ptr;

// Workgroup barrier for data in LDS only: __syncthreads() would also wait for every load and store in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Bound by the store of the spectra (8 bytes per frequency) and the transforms; the tile's samples come in as rows of
// neighbouring lanes, one row, then one column per thread is transformed in registers.  The phases of a workgroup wait for memory and
// for each other, so what counts is how many workgroups a compute unit holds (finish_geom): five waves per SIMD forward (88 to 95 registers), four inverse
// (106; three where columns of 32 make it 147), and no vector register spilled.  Scalar ones are: 13 and 31 (columns of 32) of an inverse, 218 to 324 of one that adds shares, which
// keeps 36 bytes a lane in scratch memory in two instances, as does the forward kernel for columns of 32 and clipped tiles.  Held to five waves, 96 registers, the inverse spilled
// 13 vector registers: kernel gradients of 120 x 120 maps, 24^3, 240 -> 203 us without.  Tests of mask bits and addresses that the
// compiler kept across columns cost 20 to 30 registers and most of the scalar ones.  40 maps of 64^3 in tiles of 16 x 24 x 24:
// forward 41 -> 37 us, inverse 41 -> 36 us; their kernels 27 -> 19 and 21 -> 16 us.
template <bool LONG, bool FULL>
__device__ __forceinline__ void tile_forward(float2* lds, EntryInfo* info, const TileFwd& A, int group)
{
    const TileGeom& G = A.G;
    float* lf = reinterpret_cast<float*>(lds);
    const int e0 = group * G.per_wg;
    if ((int)threadIdx.x < G.per_wg) info[threadIdx.x] = entry_info(G, e0 + threadIdx.x);
    lds_barrier();
    if (G.clip) {
        if (G.vw == 4) load_samples<4, true>(lf, A.src, G, info);
        else if (G.vw == 2) load_samples<2, true>(lf, A.src, G, info);
        else load_samples<1, true>(lf, A.src, G, info);
    } else {
        if (G.vw == 4) load_samples<4, false>(lf, A.src, G, info);
        else if (G.vw == 2) load_samples<2, false>(lf, A.src, G, info);
        else load_samples<1, false>(lf, A.src, G, info);
    }
    lds_barrier();
#define ZNN_CALL(L) rows_r2c<L, FULL>(lds, G)
    ZNN_TILE_SWITCH(LONG, G.M[2], (void)0, ZNN_CALL)
#undef ZNN_CALL
    lds_barrier();
    if (G.M[1] > 1) {
#define ZNN_CALL(L) columns_y<L, -1, FULL>(lds, G)
        ZNN_TILE_SWITCH(LONG, G.M[1], (void)0, ZNN_CALL)
#undef ZNN_CALL
        lds_barrier();
    }
#define ZNN_CALL(L) columns_z_store<L, FULL>(lds, A.dst, G, e0)
    ZNN_TILE_SWITCH(LONG, G.M[0], store_plane(lds, A.dst, G, e0), ZNN_CALL)
#undef ZNN_CALL
}

template <bool LONG, bool FULL>
__global__ void __launch_bounds__(kTileThreads, 4) k_tile_fwd(TileFwd A)
{
    extern __shared__ float2 lds[];
    __shared__ EntryInfo info[kTileEntries];
    tile_forward<LONG, FULL>(lds, info, A, blockIdx.x);
}

// Transforms of both operands of a pass in one launch, the second one's workgroups from `second` on (its tiles are not FULL).
struct TileFwdPair { TileFwd item[2]; unsigned second; };
template <bool LONG, bool FULL>
__global__ void __launch_bounds__(kTileThreads, 4) k_tile_fwd_pair(TileFwdPair P)
{
    extern __shared__ float2 lds[];
    __shared__ EntryInfo info[kTileEntries];
    if (blockIdx.x < P.second) tile_forward<LONG, FULL>(lds, info, P.item[0], blockIdx.x);
    else tile_forward<LONG, false>(lds, info, P.item[1], blockIdx.x - P.second);
}

template <bool LONG, bool SPLIT>
__device__ __forceinline__ void tile_inverse(float2* lds, EntryInfo* info, float* bias, const TileInv& A, int group)
{
    const TileGeom& G = A.G;
    const float* lf = reinterpret_cast<const float*>(lds);
    const int e0 = group * G.per_wg;
    if ((int)threadIdx.x < G.per_wg) {
        info[threadIdx.x] = entry_info(G, e0 + threadIdx.x);
        if (A.finish.y) bias[threadIdx.x] = A.finish.bias[info[threadIdx.x].map];
    }
#define ZNN_CALL(L) (load_columns_z<L, SPLIT>)(lds, A, e0)
    ZNN_TILE_SWITCH(LONG, G.M[0], load_plane(lds, A, e0), ZNN_CALL)
#undef ZNN_CALL
    lds_barrier();
    if (G.M[1] > 1) {
#define ZNN_CALL(L) columns_y<L, +1, true>(lds, G)
        ZNN_TILE_SWITCH(LONG, G.M[1], (void)0, ZNN_CALL)
#undef ZNN_CALL
        lds_barrier();
    }
#define ZNN_CALL(L) rows_c2r<L>(lds, G)
    ZNN_TILE_SWITCH(LONG, G.M[2], (void)0, ZNN_CALL)
#undef ZNN_CALL
    lds_barrier();
    if (A.finish.y || A.finish.deriv) {
        if (G.vw == 4) store_samples<4, true>(lf, A, info, bias);
        else if (G.vw == 2) store_samples<2, true>(lf, A, info, bias);
        else store_samples<1, true>(lf, A, info, bias);
    } else {
        if (G.vw == 4) store_samples<4, false>(lf, A, info, bias);
        else if (G.vw == 2) store_samples<2, false>(lf, A, info, bias);
        else store_samples<1, false>(lf, A, info, bias);
    }
}

template <bool LONG, bool SPLIT>
__global__ void __launch_bounds__(kTileThreads, LONG ? 3 : 4) k_tile_inv(TileInv A)
{
    extern __shared__ float2 lds[];
    __shared__ EntryInfo info[kTileEntries];
    __shared__ float bias[kTileEntries];
    tile_inverse<LONG, SPLIT>(lds, info, bias, A, blockIdx.x);
}

// Images and kernel gradients of one layer in one launch, the gradients' workgroups from `second` on.
struct TileInvPair { TileInv item[2]; unsigned second; };
template <bool LONG>
__global__ void __launch_bounds__(kTileThreads, LONG ? 3 : 4) k_tile_inv_pair(TileInvPair P)
{
    extern __shared__ float2 lds[];
    __shared__ EntryInfo info[kTileEntries];
    __shared__ float bias[kTileEntries];
    if (blockIdx.x < P.second) tile_inverse<LONG, false>(lds, info, bias, P.item[0], blockIdx.x);
    else tile_inverse<LONG, true>(lds, info, bias, P.item[1], blockIdx.x - P.second);
}

// gin[x] = sum over the tiles that cover x, in ascending order (overlap-add), times the rectifier's derivative if there is one below.  Bound by the read of the tiles.
struct TileAdd { const float* src; float* dst; const float* deriv; int M[3], T[3], hop[3], n[3]; FastDiv fhop[3], fnx; int xy, per_row, groups, zs; };

// tiles lo .. hi along axis d cover coordinate c
__device__ __forceinline__ void tiles_over(const TileAdd& A, int d, int c, int& lo, int& hi)
{
    hi = min((int)fdiv((unsigned)c, A.fhop[d]), A.T[d] - 1);
    const int first = c - A.M[d] + 1;                   // first tile start that still covers c
    lo = first <= 0 ? 0 : (int)fdiv((unsigned)(first + A.hop[d] - 1), A.fhop[d]);
}

// At most two tiles per axis (M <= 2 B): a thread keeps the places of its (y, x) in the four tiles of a layer of tiles --
// places that do not exist repeat one that does, with weight zero, so that no load is conditional -- and walks zs values of
// z, whose one or two layers are uniform: 520 -> 290 us for 125 tiles of 24^3 of 120 maps against one thread per voxel.
// A thread takes VW neighbouring voxels, which lie in the same tiles where lengths and hops are multiples of VW: a load of one word per lane takes as
// long as one of four.  40 maps of 64^3 30 -> 24 us, 80 of 256^2 24 -> 16; the first, of 24^3 tiles, goes at the rate of memory.
template <int VW>
__global__ void __launch_bounds__(256) k_tile_add2(TileAdd A)
{
    typedef typename VecOf<VW>::type vec;
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= A.groups) return;
    const long map = blockIdx.z;
    const int y = (int)fdiv((unsigned)u, A.fnx), x = (u - y * A.per_row) * VW, left = min(VW, A.n[2] - x);
    int blo, bhi, dlo, dhi;
    tiles_over(A, 1, y, blo, bhi);
    tiles_over(A, 2, x, dlo, dhi);
    const int vol = A.M[0] * A.M[1] * A.M[2];
    int at[4];
    float weight[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int b = min(blo + (i >> 1), bhi), d = min(dlo + (i & 1), dhi);
        at[i] = (b * A.T[2] + d) * vol + (y - b * A.hop[1]) * A.M[2] + (x - d * A.hop[2]);
        weight[i] = blo + (i >> 1) <= bhi && dlo + (i & 1) <= dhi ? 1.f : 0.f;
    }
    const long layer = (long)A.T[1] * A.T[2] * vol;
    const float* base = A.src + map * (A.T[0] * layer);
    const int z1 = min(A.n[0], ((int)blockIdx.y + 1) * A.zs);
#pragma unroll 4
    for (int z = blockIdx.y * A.zs; z < z1; ++z) {
        int lo, hi;
        tiles_over(A, 0, z, lo, hi);
        float sum[VW];
#pragma unroll
        for (int c = 0; c < VW; ++c) sum[c] = 0.f;
        auto add = [&](int tile) __attribute__((always_inline)) {
            const float* p = base + tile * layer + (z - tile * A.hop[0]) * (A.M[1] * A.M[2]);
            float v[4][VW];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const vec t = *reinterpret_cast<const vec*>(p + at[i]);
                __builtin_memcpy(v[i], &t, sizeof(vec));
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int c = 0; c < VW; ++c) sum[c] = fmaf(weight[i], v[i][c], sum[c]);
        };
        add(lo);
        if (hi > lo) add(hi);
        const long to = (map * A.n[0] + z) * (long)A.xy + y * A.n[2] + x;
        if (A.deriv) {
#pragma unroll
            for (int c = 0; c < VW; ++c)
                if (c < left) sum[c] = A.deriv[to + c] > 0.f ? sum[c] : 0.f;
        }
        if (left == VW) {
            vec t;
            __builtin_memcpy(&t, sum, sizeof(vec));
            *reinterpret_cast<vec*>(A.dst + to) = t;
        } else {
#pragma unroll
            for (int c = 0; c < VW; ++c)
                if (c < left) A.dst[to + c] = sum[c];
        }
    }
}

__global__ void __launch_bounds__(256) k_tile_add(TileAdd A)
{
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= A.xy) return;
    const int z = blockIdx.y;
    const long map = blockIdx.z;
    const int y = (int)fdiv((unsigned)u, A.fnx), x = u - y * A.n[2];
    int lo[3], hi[3];
    tiles_over(A, 0, z, lo[0], hi[0]);
    tiles_over(A, 1, y, lo[1], hi[1]);
    tiles_over(A, 2, x, lo[2], hi[2]);
    const long vol = (long)A.M[0] * A.M[1] * A.M[2];
    const float* base = A.src + map * ((long)A.T[0] * A.T[1] * A.T[2] * vol);
    float sum = 0.f;
    for (int a = lo[0]; a <= hi[0]; ++a)
        for (int b = lo[1]; b <= hi[1]; ++b)
            for (int d = lo[2]; d <= hi[2]; ++d)
                sum += base[(((long)a * A.T[1] + b) * A.T[2] + d) * vol +
                            ((z - a * A.hop[0]) * A.M[1] + (y - b * A.hop[1])) * A.M[2] + (x - d * A.hop[2])];
    const long to = (map * A.n[0] + z) * (long)A.xy + u;
    if (A.deriv) sum = A.deriv[to] > 0.f ? sum : 0.f;
    A.dst[to] = sum;
}

// ---------------------------------------------------------------- matrix products per frequency
// C[m][n] = sum_k A[m][k] B[k][n] (CONJ: conj(A)) for every frequency, on v_mfma_f32_16x16x4_f32.  A workgroup owns
// 16 MT x 16 NT results of a block of 16 frequencies, each of its NW waves 16 / NW of the frequencies (real and imaginary
// part in accumulators of their own).  A chunk of four k of both operands is copied to LDS as
// it lies in memory (runs of 16 frequencies = 128 bytes; 16 bytes per lane, no registers), S - 1 chunks ahead of the one in use:
// a workgroup waits for the oldest copies alone.  A lane reads the two frequencies of its row and k with one 16-byte access; the eight 16-byte pieces of a run are
// stored in an order that depends on the row (piece ^ (row / 2) % 8), so that sixteen rows cover all banks, and the results
// leave through LDS in the same arrangement, as full lines.  All workgroups of a block run on one XCD next to each
// other in time.
// What bounds it is the way of the operands to LDS, so it matters that copies are requested before the products they overlap: the
// scheduler had moved every second chunk's behind them, next to the wait (1190 -> 1140 us on 120 x 125 x 120 products).  16 x 16 results by eight
// waves with three buffers keep 24 waves on a unit: 80 x 144 x 80 products of 544 frequencies 53 -> 48 us (16 x 48 results by four
// waves, two buffers), 20 x 80 x 28 43 -> 38 us, 40 x 45 x 40 of 4992 59 -> 55 us.  On 120 x 125 x 120: 1245 us, and 1166 us for 32 x 32 results by four waves; of
// these alone the products take 880 us and the copies 560.  Tried for wide layers: 64 x 32 results by eight waves, three buffers, one workgroup on a unit (1190 us), 32 x 32
// with three buffers (1240 us), by eight waves with two (1210 us), 48 x 48 (1370 us).
// Tried: operands straight from global memory to the lanes of v_mfma_f32_4x4x1_16B_f32, whose sixteen blocks are the
// sixteen frequencies: neighbouring lanes then lie in different rows, 64 cache accesses per load, 3.3 ms per product
// of 96^3 images and 120 x 120 maps; the same through LDS: 1.42 ms (the short MFMAs issue at 80 % of their rate, and the
// results leave as 8-byte pieces).
struct TileProduct {
    const float2* A; const float2* B; float2* C;
    long blkA, blkB, blkC, splitC;      // elements from one frequency block (split of k) to the next
    int am, ak, bn, bk, cm, cn;         // element strides
    int M, N, K;
    int gm, gn, splits, blocks;         // workgroups along m and n of a block, splits of k, frequency blocks
    int run;                            // workgroups per XCD
};

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kChunk = 4;           // k of a chunk

// Workgroup barrier behind this wave's LDS reads and copies but the newest N.  The wait is the builtin, as the compiler has to know that the
// older copies have landed: behind a wait in inline assembly it puts one for all copies before the next LDS read.
template <int N>
__device__ __forceinline__ void copies_barrier()
{
    __builtin_amdgcn_s_waitcnt((N & 15) | (N >> 4) << 14 | 7 << 4);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int MT, int NT, int NW, int S, bool CONJ>
__device__ __forceinline__ void tile_product(const TileProduct& P, unsigned group)
{
    constexpr int RA = 16 * MT, RB = 16 * NT;               // rows of A and B in LDS
    constexpr int FP = 8 / NW;                              // pairs of frequencies of a wave
    constexpr int kBuf = (RA + RB) * kChunk * 8;
    constexpr int LA = RA * kChunk / 8 / NW, LB = RB * kChunk / 8 / NW;     // copies of 1 KiB (8 rows) per wave and chunk
    static_assert(RA * kChunk / 8 % NW == 0 && RB * kChunk / 8 % NW == 0, "");
    __shared__ float4 buf0[kBuf];
    __shared__ float4 buf1[kBuf];
    __shared__ float4 buf2[S > 2 ? kBuf : 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // consecutive workgroups go to the eight XCDs in turn: each XCD takes a contiguous run of (block, tile) pairs
    const int per = P.gm * P.gn * P.splits;
    const int id = (group & 7) * P.run + (group >> 3);
    const int blk = id / per;
    if (blk >= P.blocks) return;
    int q = id - blk * per;
    const int split = q / (P.gm * P.gn);
    q -= split * P.gm * P.gn;
    const int gi = q / P.gn, gj = q - gi * P.gn;
    const int m0 = gi * RA, n0 = gj * RB;
    const int kper = ((P.K + P.splits - 1) / P.splits + kChunk - 1) / kChunk * kChunk;
    const int k0 = split * kper, k1 = min(P.K, k0 + kper);

    const char* A = reinterpret_cast<const char*>(P.A + blk * P.blkA);
    const char* B = reinterpret_cast<const char*>(P.B + blk * P.blkB);
    // copy c of a chunk: k = c / (R / 8), rows 8 (c % (R / 8)) .. + 7; the lane fills piece slot lane % 8 of row lane / 8
    unsigned ao[LA], bo[LB];
#pragma unroll
    for (int c = 0; c < LA; ++c) {
        const int row = 8 * ((wave * LA + c) % (RA / 8)) + (lane >> 3);
        ao[c] = (unsigned)(min(m0 + row, P.M - 1) * P.am) * 8u + (unsigned)(((lane & 7) ^ ((row >> 1) & 7)) * 16);
    }
#pragma unroll
    for (int c = 0; c < LB; ++c) {
        const int row = 8 * ((wave * LB + c) % (RB / 8)) + (lane >> 3);
        bo[c] = (unsigned)(min(n0 + row, P.N - 1) * P.bn) * 8u + (unsigned)(((lane & 7) ^ ((row >> 1) & 7)) * 16);
    }
    // requested where it stands, in front of the products
    auto copy = [&](float4* buf, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < LA; ++c) {
            const int kk = min(k + (wave * LA + c) / (RA / 8), k1 - 1);
            __builtin_amdgcn_global_load_lds((global_cptr)(A + (long)kk * (P.ak * 8) + ao[c]), (lds_ptr)(buf + (wave * LA + c) * 64), 16, 0, 0);
        }
#pragma unroll
        for (int c = 0; c < LB; ++c) {
            const int kk = min(k + (wave * LB + c) / (RB / 8), k1 - 1);
            __builtin_amdgcn_global_load_lds((global_cptr)(B + (long)kk * (P.bk * 8) + bo[c]),
                                             (lds_ptr)(buf + RA * kChunk * 8 + (wave * LB + c) * 64), 16, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    f32x4 re[2 * FP][MT][NT], im[2 * FP][MT][NT];           // [frequency]
#pragma unroll
    for (int f = 0; f < 2 * FP; ++f)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int t = 0; t < NT; ++t) re[f][i][t] = im[f][i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int row = lane & 15, kl = lane >> 4;
    int at[FP];
#pragma unroll
    for (int h = 0; h < FP; ++h) at[h] = row * 8 + ((FP * wave + h) ^ (row >> 1));
    auto chunk = [&](const float4* buf, int k, auto last) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < FP; ++h) {                       // frequencies 2 h, 2 h + 1 of the wave
            const float4* pa = buf + kl * RA * 8;
            const float4* pb = buf + (RA * kChunk + kl * RB) * 8;
            float4 a[MT], b[NT];
#pragma unroll
            for (int i = 0; i < MT; ++i) a[i] = pa[i * 128 + at[h]];
#pragma unroll
            for (int t = 0; t < NT; ++t) b[t] = pb[t * 128 + at[h]];
            if constexpr (decltype(last)::value) {          // k behind the last one
                const bool in = k + kl < k1;
#pragma unroll
                for (int i = 0; i < MT; ++i) a[i] = make_float4(in ? a[i].x : 0.f, in ? a[i].y : 0.f, in ? a[i].z : 0.f, in ? a[i].w : 0.f);
            }
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const float n0_ = -a[i].y, n1_ = -a[i].w;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    f32x4 &r0 = re[2 * h][i][t], &i0 = im[2 * h][i][t], &r1 = re[2 * h + 1][i][t], &i1 = im[2 * h + 1][i][t];
                    r0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i].x, b[t].x, r0, 0, 0, 0);
                    i0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i].x, b[t].y, i0, 0, 0, 0);
                    r1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i].z, b[t].z, r1, 0, 0, 0);
                    i1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i].z, b[t].w, i1, 0, 0, 0);
                    r0 = __builtin_amdgcn_mfma_f32_16x16x4f32(CONJ ? a[i].y : n0_, b[t].y, r0, 0, 0, 0);
                    i0 = __builtin_amdgcn_mfma_f32_16x16x4f32(CONJ ? n0_ : a[i].y, b[t].x, i0, 0, 0, 0);
                    r1 = __builtin_amdgcn_mfma_f32_16x16x4f32(CONJ ? a[i].w : n1_, b[t].w, r1, 0, 0, 0);
                    i1 = __builtin_amdgcn_mfma_f32_16x16x4f32(CONJ ? n1_ : a[i].w, b[t].z, i1, 0, 0, 0);
                }
            }
        }
    };
    // never taken: tells the optimizer that LDS holds data
    if (P.K < 0) buf0[threadIdx.x] = buf1[threadIdx.x] = buf2[0] = *reinterpret_cast<const float4*>(A + threadIdx.x * 16);
    const int n = k1 > k0 ? (k1 - k0 + kChunk - 1) / kChunk : 0;            // chunks
    auto buffer = [&](auto which) -> float4* {
        constexpr int W = decltype(which)::value;
        if constexpr (W == 0) return buf0; else if constexpr (W == 1) return buf1; else return buf2;
    };
    // the first copies of a workgroup without k (an empty share) read the last k there is
    copy(buf0, k0);
    if constexpr (S > 2) copy(buf1, k0 + kChunk);
    int c = 0;
    // whole turns of the buffers; copies behind the last chunk repeat it
    auto turn = [&](auto which) __attribute__((always_inline)) {
        constexpr int W = decltype(which)::value;
        copies_barrier<(S - 2) * (LA + LB)>();
        copy(buffer(std::integral_constant<int, (W + S - 1) % S>{}), k0 + min(c + W + S - 1, n - 1) * kChunk);
        chunk(buffer(which), k0 + (c + W) * kChunk, std::false_type{});
    };
    for (; c + S < n; c += S) {
        turn(std::integral_constant<int, 0>{});
        turn(std::integral_constant<int, 1>{});
        if constexpr (S > 2) turn(std::integral_constant<int, 2>{});
    }
    // the last one to S chunks
    if (n > 0) {
        copies_barrier<0>();
        if (c + S - 1 < n) copy(buffer(std::integral_constant<int, S - 1>{}), k0 + (c + S - 1) * kChunk);
        chunk(buf0, k0 + c * kChunk, std::true_type{});
    }
    if (c + 1 < n) {
        copies_barrier<0>();
        chunk(buf1, k0 + (c + 1) * kChunk, std::true_type{});
    }
    if (S > 2 && c + 2 < n) {
        copies_barrier<0>();
        chunk(buf2, k0 + (c + 2) * kChunk, std::true_type{});
    }
    copies_barrier<0>();
    // results: lane (n = lane % 16, q = lane / 16) holds rows 4 q .. 4 q + 3 of a tile.  SR rows at a time go through LDS, through
    // the two buffers in turn.
    constexpr int SR = 8 * 8 * RB <= kBuf ? 8 : 4;
    float2* C = P.C + blk * P.blkC + split * P.splitC;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int part = 0; part < 16 / SR; ++part) {
            const int mrow = m0 + 16 * i + SR * part;
            if (mrow >= P.M) break;                                 // uniform
            float4* const buf = (i * (16 / SR) + part) & 1 ? buf1 : buf0;
            if ((lane >> 4) * 4 / SR == part) {
                const int q4 = (lane >> 4) % (SR / 4);
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float4* o = buf + ((4 * q4 + r) * RB + 16 * t) * 8;
#pragma unroll
                        for (int h = 0; h < FP; ++h)
                            o[at[h]] = make_float4(re[2 * h][i][t][r], im[2 * h][i][t][r], re[2 * h + 1][i][t][r], im[2 * h + 1][i][t][r]);
                    }
            }
            lds_barrier();
#pragma unroll 4
            for (int u = threadIdx.x; u < SR * RB * 8; u += 64 * NW) {
                const int m = u / (RB * 8), n = (u / 8) % RB, piece = (u & 7) ^ ((n >> 1) & 7);
                if (mrow + m < P.M && n0 + n < P.N)
                    *reinterpret_cast<float4*>(C + (long)(mrow + m) * P.cm + (long)(n0 + n) * P.cn + piece * 2) = buf[u];
            }
        }
}

template <int MT, int NT, int NW, int S, bool CONJ>
__global__ void __launch_bounds__(64 * NW, NW == 4 ? 2 : 6) k_tile_product(TileProduct P)
{
    tile_product<MT, NT, NW, S, CONJ>(P, blockIdx.x);
}

// The conjugated products of the backward pass and of the kernel gradient in one launch, the latter's workgroups from `second` (a
// multiple of eight) on.
struct TileProductPair { TileProduct item[2]; unsigned second; };
__global__ void __launch_bounds__(512, 6) k_tile_product_pair(TileProductPair A)
{
    const int q = blockIdx.x >= A.second;
    tile_product<1, 1, 8, 3, true>(A.item[q], blockIdx.x - (q ? A.second : 0));
}

// ---------------------------------------------------------------- launches
TileGeom base_geom(const Tiling& L)
{
    TileGeom G = {};
    for (int d = 0; d < 3; ++d) G.M[d] = L.M[d];
    G.Mxh = L.M[2] / 2 + 1;
    return G;
}

unsigned mask_of(int o, int w, int sp)
{
    unsigned m = 0;
    for (int i = 0; i < w; ++i) m |= 1u << (o + i * sp);
    return m;
}

bool has_long(const TileGeom& G) { return G.M[0] > 24 || G.M[1] > 24 || G.M[2] > 24; }

// Fills what follows from the fields set by the caller; returns threads and LDS bytes of a workgroup.  Entries per
// workgroup: as many as keep the threads of the column passes busiest within 40 KiB of LDS (three workgroups per compute
// unit or more; a single larger tile still leaves two), while the launch has two workgroups per compute unit.
void finish_geom(TileGeom& G, long entries, bool inverse, int* threads, size_t* lds, int given = 0)
{
    G.entries = (int)entries;
    if (!G.count) G.count = G.T[0] * G.T[1] * G.T[2];
    const size_t one = sizeof(float2) * (size_t)G.w[0] * G.M[1] * G.Mxh;     // the planes along z that hold samples
    const int cols = G.M[0] > 1 ? G.M[1] * G.Mxh : G.Mxh;
    int nb = 1;
    double best = 0;
    for (int c = 1; c <= kTileEntries; ++c) {
        if (c > 1 && (c * one > 40 * 1024 || (entries + c - 1) / c < 512 || c * cols > 320)) break;
        const int t = (c * cols + 63) / 64 * 64;
        const double use = (double)(c * cols) / t;
        if (use > best + 0.02) { best = use; nb = c; }
    }
    // a launch of twice the waves takes twice the entries, if that leaves enough workgroups
    if (given && nb * 2 <= kTileEntries && nb * 2 * one <= 40 * 1024 && entries >= 1024L * nb) nb *= 2;
    G.per_wg = nb;
    for (int d = 0; d < 3; ++d) {
        G.fw[d] = make_fastdiv((unsigned)G.w[d]);
        G.mask[d] = mask_of(G.o[d], G.w[d], G.sp[d]);
    }
    const int last = std::min(G.w[2], G.n[2] - (G.T[2] - 1) * G.hop[2]);        // samples per row of the last tile along x
    G.vw = G.sp[2] > 1 ? 1 : G.w[2] % 4 == 0 && last >= 4 ? 4 : G.w[2] % 2 == 0 && last >= 2 ? 2 : 1;
    G.clip = entries % nb != 0;
    for (int d = 0; d < 3; ++d) G.clip |= G.n[d] - (G.T[d] - 1) * G.hop[d] < G.w[d];
    G.fwx = make_fastdiv((unsigned)(G.w[2] / G.vw));
    G.fMxh = make_fastdiv((unsigned)G.Mxh);
    G.fcol = make_fastdiv((unsigned)(G.M[1] * G.Mxh));
    // Waves of a workgroup.  The unit places a workgroup of five waves two on one SIMD, so it holds two such workgroups where registers
    // would do for four: workgroups of four waves, or of two where no phase but the last has more rows and columns, if a unit gets three of them.
    // 40 maps of 64^3, 1800 tiles: 5 waves 40.9 / 41.4 / 39.7 us (inverse, images, gradients), 4 waves 37.5 / 39.0 / 34.6, 3 waves 40.0 / 41.5 / 35.3; kernels 5, 4, 2
    // waves 26.8, 23.3, 19.5.  Fewer workgroups leave the unit to one or two of them, and these take all the waves the column passes fill (108
    // workgroups 9.0 us, by two waves 14.8), as do tiles that fill half of its LDS (24^3: 349 us, by four waves 470).  Inverses with columns of 32 have registers for
    // twelve waves on a unit: two waves where it gets more than three workgroups, four where LDS or their number leaves it three.  2, 4 waves: three of them, 102 maps in tiles
    // of 32 x 20 x 20 115 / 91 us (14 maps 56 / 39), 102 of 16 x 32 15.4 / 12.2; four, 62 maps of 32^2 20.8 / 23.6; six and more, 90 maps of 12 x 32 x 16 84 / 104.
    const int rows = nb * G.w[0] * std::max(G.w[1], G.Mxh);         // or columns along y
    const long fit = std::min((long)(kUnitLds / (nb * one + kTileStatic)), (entries + nb * 256 - 1) / (nb * 256));
    if (fit < 3)
        *threads = std::min(kTileThreads, std::max(128, (nb * cols + 63) / 64 * 64));
    else if (rows <= 128)
        *threads = 128;
    else
        *threads = inverse && has_long(G) && fit > 3 ? 128 : 256;
    if (given) *threads = given;
    *lds = nb * one;
    G.rows_per_step = *threads / (G.w[2] / G.vw);
    G.step[2] = G.rows_per_step % G.w[1];
    G.step[1] = G.rows_per_step / G.w[1] % G.w[0];
    G.step[0] = G.rows_per_step / G.w[1] / G.w[0];
}

bool is_full(const TileGeom& G) { return G.w[0] == G.M[0] && G.w[1] == G.M[1] && G.w[2] == G.M[2]; }

// real tiles of one operand and where their spectra go
struct TileOperand { const char* name; TileGeom G; long entries; const float* src; float2* dst; };

int forward_tiles(const TileOperand& O, hipStream_t s)
{
    TileFwd A;
    int threads; size_t lds;
    A.src = O.src; A.dst = O.dst; A.G = O.G;
    finish_geom(A.G, O.entries, false, &threads, &lds);
    const dim3 grid((unsigned)((O.entries + A.G.per_wg - 1) / A.G.per_wg)), block(threads);
    const bool full = is_full(A.G);
    if (has_long(A.G)) {
        if (full) ZNN_LAUNCH(O.name, s, (k_tile_fwd<true, true>), grid, block, lds, A);
        else      ZNN_LAUNCH(O.name, s, (k_tile_fwd<true, false>), grid, block, lds, A);
    } else {
        if (full) ZNN_LAUNCH(O.name, s, (k_tile_fwd<false, true>), grid, block, lds, A);
        else      ZNN_LAUNCH(O.name, s, (k_tile_fwd<false, false>), grid, block, lds, A);
    }
    return check_launch(O.name);
}

// Both operands of a pass.  Neither waits for the other, and the launch of the smaller one would not fill the chip: 20 -> 28 maps, 23 x 131 x 115,
// forward 38.8 + 14.6 us and gradient 38.7 + 46.6 in launches of their own; a round 422 -> 391 us, one of the 2D net 422 -> 394.
int forward_tiles(const char* name, const TileOperand& first, const TileOperand& second, hipStream_t s)
{
    const TileOperand* const O[2] = {&first, &second};
    TileFwdPair P;
    int threads[2]; size_t lds[2]; unsigned groups[2];
    for (int q = 0; q < 2; ++q) {
        P.item[q].src = O[q]->src; P.item[q].dst = O[q]->dst; P.item[q].G = O[q]->G;
        finish_geom(P.item[q].G, O[q]->entries, false, &threads[q], &lds[q]);
    }
    const int most = std::max(threads[0], threads[1]);
    for (int q = 0; q < 2; ++q) {
        if (threads[q] < most) {
            P.item[q].G = O[q]->G;
            finish_geom(P.item[q].G, O[q]->entries, false, &threads[q], &lds[q], most);
        }
        groups[q] = (unsigned)((O[q]->entries + P.item[q].G.per_wg - 1) / P.item[q].G.per_wg);
    }
    P.second = groups[0];
    const dim3 grid(groups[0] + groups[1]), block(most);
    const size_t bytes = std::max(lds[0], lds[1]);
    const bool full = is_full(first.G);
    if (has_long(first.G)) {
        if (full) ZNN_LAUNCH(name, s, (k_tile_fwd_pair<true, true>), grid, block, bytes, P);
        else      ZNN_LAUNCH(name, s, (k_tile_fwd_pair<true, false>), grid, block, bytes, P);
    } else {
        if (full) ZNN_LAUNCH(name, s, (k_tile_fwd_pair<false, true>), grid, block, bytes, P);
        else      ZNN_LAUNCH(name, s, (k_tile_fwd_pair<false, false>), grid, block, bytes, P);
    }
    return check_launch(name);
}

// spectra (partial sums of them, to be added) and where the real tiles go
struct TileResult { TileGeom G; long entries; const float2* src; float* dst; float scale; int splits; long split_stride; Finish finish; };

TileInv inverse_of(const TileResult& R, int given, int* threads, size_t* lds, unsigned* groups)
{
    TileInv A;
    A.G = R.G;
    finish_geom(A.G, R.entries, true, threads, lds, given);
    A.src = R.src; A.dst = R.dst; A.scale = R.scale; A.splits = R.splits; A.split_stride = R.split_stride; A.finish = R.finish;
    *groups = (unsigned)((R.entries + A.G.per_wg - 1) / A.G.per_wg);
    return A;
}

int inverse_tiles(const char* name, const TileResult& R, hipStream_t s)
{
    int threads; size_t lds; unsigned groups;
    const TileInv A = inverse_of(R, 0, &threads, &lds, &groups);
    const dim3 grid(groups), block(threads);
    if (has_long(A.G)) {
        if (A.splits > 1) ZNN_LAUNCH(name, s, (k_tile_inv<true, true>), grid, block, lds, A);
        else              ZNN_LAUNCH(name, s, (k_tile_inv<true, false>), grid, block, lds, A);
    } else {
        if (A.splits > 1) ZNN_LAUNCH(name, s, (k_tile_inv<false, true>), grid, block, lds, A);
        else              ZNN_LAUNCH(name, s, (k_tile_inv<false, false>), grid, block, lds, A);
    }
    return check_launch(name);
}

// Two results of one tiling, the first one not in shares.
int inverse_tiles(const char* name, const TileResult& first, const TileResult& second, hipStream_t s)
{
    TileInvPair P;
    const TileResult* const R[2] = {&first, &second};
    int threads[2]; size_t lds[2]; unsigned groups[2];
    for (int q = 0; q < 2; ++q) P.item[q] = inverse_of(*R[q], 0, &threads[q], &lds[q], &groups[q]);
    const int most = std::max(threads[0], threads[1]);
    for (int q = 0; q < 2; ++q)
        if (threads[q] < most) P.item[q] = inverse_of(*R[q], most, &threads[q], &lds[q], &groups[q]);
    P.second = groups[0];
    const dim3 grid(groups[0] + groups[1]), block(most);
    const size_t bytes = std::max(lds[0], lds[1]);
    if (has_long(first.G)) ZNN_LAUNCH(name, s, k_tile_inv_pair<true>, grid, block, bytes, P);
    else                   ZNN_LAUNCH(name, s, k_tile_inv_pair<false>, grid, block, bytes, P);
    return check_launch(name);
}

// Workgroups of a product with MT x NT tiles of 16 x 16 results each, a multiple of eight.
long place_groups(TileProduct& P, int MT, int NT)
{
    P.gm = (P.M + 16 * MT - 1) / (16 * MT);
    P.gn = (P.N + 16 * NT - 1) / (16 * NT);
    const long run = ((long)P.blocks * P.gm * P.gn * P.splits + 7) / 8;
    P.run = (int)std::min(run, 2147483647L / 8);
    return run * 8;
}

template <int MT, int NT, int NW, int S>
int product_of(const char* name, bool conj, TileProduct P, hipStream_t s)
{
    const long grid = place_groups(P, MT, NT);
    if (grid >= 2147483647L) return fail(ZNN_EUNSUPPORTED, "too many tiles for one launch");
    if (conj) ZNN_LAUNCH(name, s, (k_tile_product<MT, NT, NW, S, true>), dim3((unsigned)grid), dim3(64 * NW), 0, P);
    else      ZNN_LAUNCH(name, s, (k_tile_product<MT, NT, NW, S, false>), dim3((unsigned)grid), dim3(64 * NW), 0, P);
    return check_launch(name);
}

// Tiles of 32 x 32 results read half as much, but a compute unit holds two of their workgroups, so they take products of at least four rounds
// of these, where padding to 32 costs little: 120 x 125 x 120 products of 7488 frequencies 1166 us against 1245, 111 x 64 x 21 187 against 207.
// Below, 16 x 16: 80 x 144 x 80 of 544 frequencies 48 us against 60, 28 x 56 x 20 of 6336 35 against 42, 40 x 45 x 40 of 4992 58 against 91.  On 177 products
// of 60 layers the rule is within 2 % of the faster one of seven shapes.
double groups_of(const TileProduct& P, int rows)
{
    return (double)P.blocks * P.splits * ((P.M + rows - 1) / rows) * ((P.N + rows - 1) / rows);
}

bool is_wide(const TileProduct& P) { return groups_of(P, 32) >= 2048 && groups_of(P, 16) >= 3.2 * groups_of(P, 32); }

int product(const char* name, bool conj, const TileProduct& P, hipStream_t s)
{
    return is_wide(P) ? product_of<2, 2, 4, 2>(name, conj, P, s) : product_of<1, 1, 8, 3>(name, conj, P, s);
}

int products(const char* name, const TileProduct& first, const TileProduct& second, hipStream_t s)
{
    TileProductPair A;
    A.item[0] = first; A.item[1] = second;
    const long grid[2] = {place_groups(A.item[0], 1, 1), place_groups(A.item[1], 1, 1)};
    if (grid[0] + grid[1] >= 2147483647L) return fail(ZNN_EUNSUPPORTED, "too many tiles for one launch");
    A.second = (unsigned)grid[0];
    ZNN_LAUNCH(name, s, k_tile_product_pair, dim3((unsigned)(grid[0] + grid[1])), dim3(512), 0, A);
    return check_launch(name);
}

constexpr int kLengths[] = {8, 12, 16, 20, 24, 32};

size_t spectra_of(const Tiling& L, long entries) { return align256(sizeof(float2) * 16 * (size_t)L.blocks * entries); }

}  // namespace

// ---------------------------------------------------------------- the tiling of a layer
// Seconds that a training round spends on tiles: transforms at 3.0 (forward) and 2.6 TB/s (inverse) of spectra, products at 4.5 TB/s and
// 110 TFLOP/s (result tiles of 16 x 16), the sum of overlapping tiles at 4.2 TB/s.  These are rates of earlier kernels on layers that fill the chip.  Of 306 rounds on the present
// ones, 4 us a launch included, it says 0.85 times the measured time at the median below 100 us (0.59 to 1.14), 0.90 to 200 us (0.65 to 1.28) and 1.02 above (0.64 to 1.32).  Node spectra count one and a half times: rounds with and without memoized ones.
static double round_seconds(const Geom& g, const Tiling& L)
{
    auto up16 = [](double v) { return std::ceil(v / 16.0) * 16.0; };
    const double w = 8.0 * 16.0 * L.blocks, T = L.tiles, nodes = g.f + g.fo, pairs = (double)g.f * g.fo;
    const double vol = (double)L.M[0] * L.M[1] * L.M[2];
    const double transforms = w * (1.5 * T * nodes / 3.0e12 + T * nodes / 2.6e12 + 1.5 * pairs / 3.3e12 + pairs / 3.0e12);
    const double products = w * (3.0 * pairs + 3.0 * T * nodes) / 4.5e12 +
                            w * (up16(g.fo) * up16(T) * g.f + up16(g.f) * up16(T) * g.fo + up16(g.f) * up16(g.fo) * T) / 110e12;
    const double sum = T > 1 ? 8.0 * vol * T * g.f / 4.2e12 : 0.0;
    return transforms + products + sum;
}

Tiling tile_search(const Geom& g, size_t spectra_bytes)
{
    Tiling best = {};
    if (g.f > 65535) return best;       // maps are an extent of the grid that sums tiles
    const int n[3] = {g.nz, g.ny, g.nx}, o[3] = {g.oz, g.oy, g.ox};
    const int S[3] = {g.spz * (g.kz - 1) + 1, g.spy * (g.ky - 1) + 1, g.spx * (g.kx - 1) + 1};
    double best_t = 0;
    auto lengths = [&](int d, int* out) {
        int c = 0;
        if (d < 2 && n[d] == 1) { out[c++] = 1; return c; }
        for (int M : kLengths)
            if (M >= S[d]) {
                out[c++] = M;
                if (M - S[d] + 1 >= o[d]) break;     // one tile covers the axis: a longer one is only padding
            }
        return c;
    };
    int lz[8], ly[8], lx[8];
    const int cz = lengths(0, lz), cy = lengths(1, ly), cx = lengths(2, lx);
    for (int a = 0; a < cz; ++a)
        for (int b = 0; b < cy; ++b)
            for (int c = 0; c < cx; ++c) {
                Tiling L = {};
                const int M[3] = {lz[a], ly[b], lx[c]};
                L.on = true;
                long T = 1;
                for (int d = 0; d < 3; ++d) {
                    L.M[d] = M[d];
                    L.B[d] = M[d] - S[d] + 1;
                    L.T[d] = (o[d] + L.B[d] - 1) / L.B[d];
                    T *= L.T[d];
                }
                const long omega = (long)M[0] * M[1] * (M[2] / 2 + 1);
                if (omega * (long)sizeof(float2) > (long)kTileLds) continue;
                // BlockOffsets counts on planes of a multiple of 4 frequencies: volumes of one row per plane stay whole
                if (M[0] > 1 && M[1] * (M[2] / 2 + 1) % 4 != 0) continue;
                L.tiles = (int)T;
                L.blocks = (int)((omega + 15) / 16);
                // entries are counted in 32 bits and an operand of a frequency block is addressed with 32-bit byte offsets
                const double most = std::max((double)T * std::max(g.f, g.fo), (double)g.f * g.fo);
                if (most >= 3e7 || (M[1] * (M[2] / 2 + 1) / 16 + 2) * most * 128.0 >= 4294967296.0) continue;
                if (tile_kernel_bytes(g, L) > spectra_bytes) continue;
                const double t = round_seconds(g, L);
                if (best_t == 0 || t < best_t) { best = L; best_t = t; }
            }
    best.seconds = best_t;
    return best;
}

size_t tile_kernel_bytes(const Geom& g, const Tiling& L) { return spectra_of(L, (long)g.f * g.fo); }
size_t tile_node_bytes(const Geom&, const Tiling& L, int maps) { return spectra_of(L, (long)maps * L.tiles); }

// splits of the tile index in the kernel gradient: enough waves to fill the chip
static int gradient_splits(const Geom& g, const Tiling& L)
{
    const long waves = (long)L.blocks * ((g.f + 15) / 16) * ((g.fo + 15) / 16);
    const int most = std::max(1, L.tiles / 16);
    return (int)std::max(1L, std::min((long)std::min(most, 16), 2048 / std::max(1L, waves)));
}

// real tiles of the backward pass before their overlapping parts are summed
static size_t add_bytes(const Tiling& L, int maps)
{
    if (L.tiles == 1) return 0;     // nothing overlaps: the inverse transform writes the result itself
    return align256(sizeof(float) * (size_t)L.M[0] * L.M[1] * L.M[2] * L.tiles * maps);
}

size_t tile_workspace_bytes(const Geom& g, const Tiling& L, int pass, bool resident)
{
    if (pass == ZNN_PASS_WGRAD)
        return tile_node_bytes(g, L, g.f) + tile_node_bytes(g, L, g.fo) + gradient_splits(g, L) * tile_kernel_bytes(g, L);
    const int outs = pass == ZNN_PASS_FWD ? g.fo : g.f;
    const size_t operands = tile_node_bytes(g, L, pass == ZNN_PASS_FWD ? g.f : g.fo) + (resident ? 0 : tile_kernel_bytes(g, L));
    // the real tiles of the backward pass take the place of the operands (see tile_bwd)
    return tile_node_bytes(g, L, outs) + std::max(operands, pass == ZNN_PASS_BWD ? add_bytes(L, outs) : 0);
}

static TileOperand tile_kernels(const Geom& g, const Tiling& L, const float* w, float2* What)
{
    TileGeom G = base_geom(L);
    const int k[3] = {g.kz, g.ky, g.kx}, sp[3] = {g.spz, g.spy, g.spx};
    for (int d = 0; d < 3; ++d) { G.T[d] = 1; G.hop[d] = 0; G.n[d] = G.w[d] = k[d]; G.o[d] = 0; G.sp[d] = sp[d]; }
    return TileOperand{"fft of kernels (tiles)", G, (long)g.f * g.fo, w, What};
}

int tile_kernel_spectra(const Geom& g, const Tiling& L, const float* w, float2* What, hipStream_t s)
{
    return forward_tiles(tile_kernels(g, L, w, What), s);
}

static TileOperand tile_images(const Geom& g, const Tiling& L, const float* in, float2* U, int first, int count)
{
    TileGeom G = base_geom(L);
    G.first = first; G.count = count;
    const int n[3] = {g.nz, g.ny, g.nx};
    for (int d = 0; d < 3; ++d) { G.T[d] = L.T[d]; G.hop[d] = L.B[d]; G.n[d] = n[d]; G.w[d] = L.M[d]; G.o[d] = 0; G.sp[d] = 1; }
    return TileOperand{"fft of image tiles", G, (long)g.f * count, in, U};
}

static TileOperand tile_gradients(const Geom& g, const Tiling& L, const float* gout, float2* V)
{
    TileGeom G = base_geom(L);
    const int o[3] = {g.oz, g.oy, g.ox};
    for (int d = 0; d < 3; ++d) {
        G.T[d] = L.T[d]; G.hop[d] = L.B[d]; G.n[d] = o[d]; G.w[d] = L.B[d]; G.o[d] = L.M[d] - L.B[d]; G.sp[d] = 1;
    }
    return TileOperand{"fft of gradient tiles", G, (long)g.fo * L.tiles, gout, V};
}

static float inv_volume(const Tiling& L) { return (float)(1.0 / ((double)L.M[0] * L.M[1] * L.M[2])); }

// The tiles come in as few equal groups as the workspace allows: one in tile_workspace_bytes, more in the built-in array of
// znn_conv3d_fwd_static.  Tiles of the forward pass do not meet, and a product adds in the same order whatever the group,
// so the results are the same bits.
int tile_fwd(const Geom& g, const Tiling& L, const float* in, const KernelSpectra& K, float* out,
             void* ws, size_t ws_bytes, float2* memo_in, const Finish& finish, hipStream_t s)
{
    const size_t kernels = K.held || K.made ? 0 : tile_kernel_bytes(g, L);
    auto image_bytes = [&](int c) { return memo_in ? 0 : spectra_of(L, (long)g.f * c); };
    int count = 0;
    for (int n = 1; n <= L.tiles && !count; ++n) {
        const int c = (L.tiles + n - 1) / n;
        if (image_bytes(c) + kernels + spectra_of(L, (long)g.fo * c) <= ws_bytes) count = c;
    }
    if (!count) return fail(ZNN_EWORKSPACE, "workspace too small for the spectra of the kernels and of one tile");
    float2* const U = memo_in ? memo_in : (float2*)ws;
    float2* const own = (float2*)((char*)ws + image_bytes(count));
    float2* const result = (float2*)((char*)own + kernels);
    float2* const made = K.made ? K.made : own;
    const float2* const What = K.held ? K.held : made;
    TileGeom G = base_geom(L);
    const int o[3] = {g.oz, g.oy, g.ox};
    for (int d = 0; d < 3; ++d) {
        G.T[d] = L.T[d]; G.hop[d] = L.B[d]; G.n[d] = o[d]; G.w[d] = L.B[d]; G.o[d] = L.M[d] - L.B[d]; G.sp[d] = 1;
    }
    for (int first = 0; first < L.tiles; first += count) {
        const int c = std::min(count, L.tiles - first);
        int rc = ZNN_OK;
        // a memo buffer takes the spectra of all tiles
        const bool transform = !memo_in || first == 0;
        const TileOperand images = memo_in ? tile_images(g, L, in, U, 0, L.tiles) : tile_images(g, L, in, U, first, c);
        if (!K.held && first == 0) rc = forward_tiles("fft of image tiles and kernels", images, tile_kernels(g, L, K.w, made), s);
        else if (transform) rc = forward_tiles(images, s);
        if (rc != ZNN_OK) return rc;
        const int tiles = memo_in ? L.tiles : c;                // of a map of U
        TileProduct P = {};
        P.A = What; P.am = g.f * 16; P.ak = 16; P.blkA = (long)g.f * g.fo * 16;
        P.B = U + (memo_in ? (long)first * 16 : 0); P.bk = tiles * 16; P.bn = 16; P.blkB = (long)g.f * tiles * 16;
        P.C = result; P.cm = c * 16; P.cn = 16; P.blkC = (long)g.fo * c * 16;
        P.M = g.fo; P.N = c; P.K = g.f; P.blocks = L.blocks; P.splits = 1;
        rc = product("spectral products forward (tiles)", false, P, s);
        G.first = first; G.count = c;
        if (rc == ZNN_OK)
            rc = inverse_tiles("inverse fft of image tiles", TileResult{G, (long)g.fo * c, result, out, inv_volume(L), 1, 0, finish}, s);
        if (rc != ZNN_OK) return rc;
    }
    return ZNN_OK;
}

static TileProduct backward_product(const Geom& g, const Tiling& L, const float2* What, const float2* V, float2* result)
{
    TileProduct P = {};
    P.A = What; P.am = 16; P.ak = g.f * 16; P.blkA = (long)g.f * g.fo * 16;
    P.B = V; P.bk = L.tiles * 16; P.bn = 16; P.blkB = (long)g.fo * L.tiles * 16;
    P.C = result; P.cm = L.tiles * 16; P.cn = 16; P.blkC = (long)g.f * L.tiles * 16;
    P.M = g.f; P.N = L.tiles; P.K = g.fo; P.blocks = L.blocks; P.splits = 1;
    return P;
}

static TileProduct gradient_product(const Geom& g, const Tiling& L, const float2* U, const float2* V, float2* sums)
{
    TileProduct P = {};
    P.splits = gradient_splits(g, L);
    P.A = U; P.am = L.tiles * 16; P.ak = 16; P.blkA = (long)g.f * L.tiles * 16;
    P.B = V; P.bn = L.tiles * 16; P.bk = 16; P.blkB = (long)g.fo * L.tiles * 16;
    P.C = sums; P.cm = 16; P.cn = g.f * 16; P.blkC = (long)g.f * g.fo * 16;
    P.splitC = P.blkC * L.blocks;
    P.M = g.f; P.N = g.fo; P.K = L.tiles; P.blocks = L.blocks;
    return P;
}

static TileResult gradient_result(const Geom& g, const Tiling& L, const TileProduct& P, float* gw)
{
    TileGeom G = base_geom(L);
    const int k[3] = {g.kz, g.ky, g.kx}, sp[3] = {g.spz, g.spy, g.spx};
    for (int d = 0; d < 3; ++d) { G.T[d] = 1; G.hop[d] = 0; G.n[d] = G.w[d] = k[d]; G.o[d] = 0; G.sp[d] = sp[d]; }
    return TileResult{G, (long)g.f * g.fo, P.C, gw, inv_volume(L), P.splits, P.splitC, Finish{}};
}

// Products of a small layer leave most of the chip idle and cost what a launch does (8 us on 40 maps x 12 tiles): joined while both together are
// at most two fills of it (a unit holds three of their workgroups).  2D nets, a round with no layer joined, those of one fill, those of two: 48^2 patch, 40 maps
// 387 us, -, 344; 64^2 430, 399, 386; 64 maps 529, 529, 476.  Layers that fill the chip by themselves keep the shape of workgroup that is best for each.
size_t tile_joined_bytes(const Geom& g, const Tiling& L)
{
    const TileProduct P = backward_product(g, L, nullptr, nullptr, nullptr), Q = gradient_product(g, L, nullptr, nullptr, nullptr);
    if (is_wide(P) || is_wide(Q) || groups_of(P, 16) + groups_of(Q, 16) > 2 * 768) return 0;
    return add_bytes(L, g.f) + tile_node_bytes(g, L, g.f) + Q.splits * tile_kernel_bytes(g, L);
}

int tile_bwd(const Geom& g, const Tiling& L, const float* gout, const KernelSpectra& K, float* gin,
             void* ws, float2* memo_gout, const Finish& finish, const TileGrad& grad, hipStream_t s)
{
    char* p = (char*)ws;
    float2* V = memo_gout;
    if (!V) { V = (float2*)p; p += tile_node_bytes(g, L, g.fo); }
    float2* made = K.made;
    if (!K.held && !made) { made = (float2*)p; p += tile_kernel_bytes(g, L); }
    const float2* const What = K.held ? K.held : made;
    int rc = K.held ? forward_tiles(tile_gradients(g, L, gout, V), s)
                    : forward_tiles("fft of gradient tiles and kernels", tile_gradients(g, L, gout, V), tile_kernels(g, L, K.w, made), s);
    if (rc != ZNN_OK) return rc;
    const bool one = L.tiles == 1;
    // The real tiles of the result take the start of the workspace, over the operands that lie there and have been
    // used by then; its spectra lie behind both.
    float* const tiles = (float*)ws;
    float2* const result = (float2*)std::max(p, (char*)ws + add_bytes(L, g.f));
    const int n[3] = {g.nz, g.ny, g.nx};
    const TileProduct P = backward_product(g, L, What, V, result);
    TileGeom G = base_geom(L);
    for (int d = 0; d < 3; ++d) {
        G.T[d] = 1; G.hop[d] = 0; G.o[d] = 0; G.sp[d] = 1;
        G.n[d] = G.w[d] = one ? n[d] : L.M[d];
    }
    const TileResult R = {G, (long)g.f * L.tiles, result, one ? gin : tiles, inv_volume(L), 1, 0, one ? finish : Finish{}};
    if (grad.gw) {
        const TileProduct Q = gradient_product(g, L, grad.U, V, (float2*)((char*)result + tile_node_bytes(g, L, g.f)));
        rc = products("spectral products backward and of gradient (tiles)", P, Q, s);
        if (rc == ZNN_OK)
            rc = inverse_tiles("inverse fft of gradient tiles and kernel gradients", R, gradient_result(g, L, Q, grad.gw), s);
    } else {
        rc = product("spectral products backward (tiles)", true, P, s);
        if (rc == ZNN_OK) rc = inverse_tiles("inverse fft of gradient tiles", R, s);
    }
    if (rc != ZNN_OK || one) return rc;
    TileAdd A = {};
    A.src = tiles; A.dst = gin; A.deriv = finish.deriv;
    for (int d = 0; d < 3; ++d) {
        A.M[d] = L.M[d]; A.T[d] = L.T[d]; A.hop[d] = L.B[d]; A.n[d] = n[d];
        A.fhop[d] = make_fastdiv((unsigned)L.B[d]);
    }
    A.xy = g.ny * g.nx;
    bool two = true;
    for (int d = 0; d < 3; ++d) two = two && L.M[d] <= 2 * L.B[d];
    const int vw = !two ? 1 : L.M[2] % 4 == 0 && L.B[2] % 4 == 0 ? 4 : L.M[2] % 2 == 0 && L.B[2] % 2 == 0 ? 2 : 1;
    A.per_row = (g.nx + vw - 1) / vw;
    A.groups = g.ny * A.per_row;
    A.fnx = make_fastdiv((unsigned)A.per_row);
    const unsigned blocks = (unsigned)((A.groups + 255) / 256);
    // z values per workgroup: few enough for four workgroups per compute unit
    A.zs = two ? (int)std::max(1L, std::min(16L, (long)blocks * g.f * g.nz / 1024)) : 1;
    const dim3 grid(blocks, (unsigned)((g.nz + A.zs - 1) / A.zs), (unsigned)g.f);
    if (!two)         ZNN_LAUNCH("sum of overlapping tiles", s, k_tile_add, grid, dim3(256), 0, A);
    else if (vw == 4) ZNN_LAUNCH("sum of overlapping tiles", s, k_tile_add2<4>, grid, dim3(256), 0, A);
    else if (vw == 2) ZNN_LAUNCH("sum of overlapping tiles", s, k_tile_add2<2>, grid, dim3(256), 0, A);
    else              ZNN_LAUNCH("sum of overlapping tiles", s, k_tile_add2<1>, grid, dim3(256), 0, A);
    return check_launch("sum of overlapping tiles");
}

int tile_wgrad_from_spectra(const Geom& g, const Tiling& L, const float2* U, const float2* V, float* gw, void* scratch,
                            hipStream_t s)
{
    const TileProduct P = gradient_product(g, L, U, V, (float2*)scratch);
    const int rc = product("spectral products of the kernel gradient (tiles)", true, P, s);
    if (rc != ZNN_OK) return rc;
    return inverse_tiles("inverse fft of kernel gradients (tiles)", gradient_result(g, L, P, gw), s);
}

int tile_wgrad(const Geom& g, const Tiling& L, const float* in, const float* gout, float* gw, void* ws, hipStream_t s)
{
    char* p = (char*)ws;
    float2* U = (float2*)p; p += tile_node_bytes(g, L, g.f);
    float2* V = (float2*)p; p += tile_node_bytes(g, L, g.fo);
    const int rc = forward_tiles("fft of image and gradient tiles", tile_images(g, L, in, U, 0, L.tiles), tile_gradients(g, L, gout, V), s);
    if (rc != ZNN_OK) return rc;
    return tile_wgrad_from_spectra(g, L, U, V, gw, p, s);
}

}  // namespace znn
