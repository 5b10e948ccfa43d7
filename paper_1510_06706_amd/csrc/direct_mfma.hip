// Direct method on the fp32 matrix cores: forward and backward pass as an
// implicit GEMM whose reduction runs over (fan-in x kernel volume), i.e. the
// sum over the edges converging on a node is part of the GEMM's K loop.  The
// kernel is in direct_mfma_impl.h; this file holds the weight packer, the
// search for the workgroup's output box and the launch.  The backward pass is
// the same contraction with the roles of the two node sets swapped, the kernel
// reflected and the output gradient zero-extended by k-1 on every side
// (Section 3.1), which the halo loader and the weight packer provide; no
// separate kernel is needed.
// Layers with more than four input-side maps take the kernel on split operands instead (direct_split.hip).
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#include "direct_mfma_tail_impl.h"
#include "direct_split.h"
#include "direct_split_impl.h"

namespace znn {

namespace {

using conv::ConvFn;
using conv::ConvTile;

constexpr int kMaxTaps = 4096;

// Packs w[f'][f][k] for the kernel of direct_mfma_tail_impl.h: per (map group, chunk, tap) the NJ x 64 operands of
// the full tiles (lane l of tile jt: output-side map jt*16 + l%16, input-side map chunk*4 + l/16), then, with
// `tail`, [8 maps][4 input maps] for the 8-map block.  For the backward pass the two map indices trade places
// and the tap is reflected.
// Several layers and passes at a time (PackArgs): the weights of a round take one launch instead of one per convolution.
// N = 1 serves the calls of a single layer, whose launch then carries 80 bytes of arguments instead of 2 KB.  Bound by the
// integer divisions of the element's number; they are 64 bits wide only where the number is.
constexpr int kPackItems = 24;
template <int N> struct PackArgs { PackItem item[N]; unsigned first[N]; int n; };

// Weights for the split kernel: a thread makes the three parts of eight input maps' weights at one tap, [group][chunk][step]
// [16-map tile][part][lane].  The leading part of a number that would round to infinity is cut instead, and an infinity or
// NaN has no other parts, so that the parts always add up to the weight.
__device__ __forceinline__ void pack_split(const PackItem& P, long t)
{
    const int taps = P.kz * P.ky * P.kx, steps = (taps + split::kTaps - 1) / split::kTaps;
    const int lane = (int)(t & 63);
    long r = t >> 6;
    const int jt = (int)(r % P.NJ); r /= P.NJ;
    const int s = (int)(r % steps); r /= steps;
    const int ic = (int)(r % P.nchunk), jg = (int)(r / P.nchunk);
    const int m = (jg * P.NJ + jt) * 16 + (lane & 15), tap = s * split::kTaps + (lane >> 4);
    const int fM = P.backward ? P.f : P.fo, fK = P.backward ? P.fo : P.f;
    float v[8];
    split::uintx4 part[3];
    bool odd = false;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int k = ic * split::kMaps + e;
        v[e] = 0.f;
        if (m < fM && k < fK && tap < taps)
            v[e] = P.backward ? P.w[((long)k * P.f + m) * taps + (taps - 1 - tap)] : P.w[((long)m * P.f + k) * taps + tap];
        odd = odd || !(fabsf(v[e]) < 3.38e38f);
    }
    if (!odd) {
#pragma unroll
        for (int p = 0; p < 3; ++p) part[p] = split::take_part8(v);
    } else {
        part[0] = part[1] = part[2] = split::uintx4{0u, 0u, 0u, 0u};
        for (int e = 0; e < 8; ++e) {
            float x = v[e];
            for (int p = 0; p < 3; ++p) {
                unsigned u = __builtin_bit_cast(unsigned, x);
                if (x != x) u |= 0x400000u;                                                 // stays a NaN
                u &= 0xffff0000u;
                part[p][e >> 1] |= e & 1 ? u : u >> 16;
                x = fabsf(x) <= 3.4028234e38f ? x - __builtin_bit_cast(float, u) : 0.f;
            }
        }
    }
    split::uintx4* out = reinterpret_cast<split::uintx4*>(P.wp) + (t >> 6) * 3 * 64 + lane;
#pragma unroll
    for (int p = 0; p < 3; ++p) out[p * 64] = part[p];
}

template <int N>
__global__ void __launch_bounds__(256) k_pack_weights(PackArgs<N> A)
{
    int q = 0;
    if (N > 1) while (q + 1 < A.n && blockIdx.x >= A.first[q + 1]) ++q;        // uniform
    const PackItem& P = A.item[q];
    const int taps = P.kz * P.ky * P.kx;
    const int WT = P.NJ * 64 + (P.tail ? conv::kTailPacked : 0);
    const long t = (long)(blockIdx.x - A.first[q]) * 256 + threadIdx.x;
    if (t >= P.total) return;
    if (P.split) { pack_split(P, t); return; }      // uniform
    int e, tap, ic, jg;
    auto place = [&](auto n) {
        e = (int)(n % (unsigned)WT); n /= (unsigned)WT;
        tap = (int)(n % (unsigned)taps); n /= (unsigned)taps;
        ic = (int)(n % (unsigned)P.nchunk);
        jg = (int)(n / (unsigned)P.nchunk);
    };
    if (P.total <= 4294967295L) place((unsigned)t);         // uniform
    else place((unsigned long)t);
    int m, k;
    if (e < P.NJ * 64) {
        m = (jg * P.NJ + e / 64) * 16 + (e & 15);
        k = ic * 4 + ((e & 63) >> 4);
    } else {
        m = P.NJ * 16 + (e - P.NJ * 64) / 4;
        k = ic * 4 + (e & 3);
    }
    const int fM = P.backward ? P.f : P.fo, fK = P.backward ? P.fo : P.f;
    float v = 0.f;
    if (m < fM && k < fK) {
        if (!P.backward) {
            v = P.w[((long)m * P.f + k) * taps + tap];
        } else {
            const int c = tap % P.kx, b = (tap / P.kx) % P.ky, a = tap / (P.kx * P.ky);
            const int rt = ((P.kz - 1 - a) * P.ky + (P.ky - 1 - b)) * P.kx + (P.kx - 1 - c);
            v = P.w[((long)k * P.f + m) * taps + rt];
        }
    }
    P.wp[t] = v;
}

__global__ void __launch_bounds__(256)
k_conv_reduce(const float* __restrict__ partial, float* __restrict__ dst, long count, int splits)
{
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    if (t >= count) return;
    float acc = partial[t];
    for (int s = 1; s < splits; ++s) acc += partial[(long)s * count + t];
    dst[t] = acc;
}

// Taps along x are walked in groups of U (direct_mfma_impl.h): the widest divisor of the
// kernel width that has an instance; 1 for sparse taps.
int group_width(int kx, int spx)
{
    if (tuning().conv_u1 || spx != 1) return 1;
    const int widths[6] = {11, 7, 5, 4, 3, 2};
    for (int i = 0; i < 6; ++i)
        if (kx % widths[i] == 0) return widths[i];
    return 1;
}

ConvFn pick_tail_kernel(int U, int nj, int nv, bool wl)
{
    switch (U) {
        case 1: return conv_tail_kernel_u1(nj, nv, wl);
        case 2: return conv_tail_kernel_u2(nj, nv, wl);
        case 3: return conv_tail_kernel_u3(nj, nv, wl);
        case 4: return conv_tail_kernel_u4(nj, nv, wl);
        case 5: return conv_tail_kernel_u5(nj, nv, wl);
        case 7: return conv_tail_kernel_u7(nj, nv, wl);
        case 11: return conv_tail_kernel_u11(nj, nv, wl);
    }
    return nullptr;
}

// The last 1..8 of the output-side maps as an 8-map block instead of a padded 16-row tile: one
// workgroup must hold all maps, and a lane's byte offset over the chunk's four source maps must fit
// 32 bits.
bool tail_applies(int fM, long svol)
{
    const int r = fM % 16;
    return !tuning().conv_no_tail && fM > 16 && fM / 16 <= 7 && r >= 1 && r <= conv::kTailMaps && svol * 16 < (1L << 32);
}

ConvFn pick_plain_kernel(int U, int nj, int nv, bool wl)
{
    switch (U) {
        case 1: return conv_plain_kernel_u1(nj, nv, wl);
        case 2: return conv_plain_kernel_u2(nj, nv, wl);
        case 3: return conv_plain_kernel_u3(nj, nv, wl);
        case 4: return conv_plain_kernel_u4(nj, nv, wl);
        case 5: return conv_plain_kernel_u5(nj, nv, wl);
        case 7: return conv_plain_kernel_u7(nj, nv, wl);
        case 11: return conv_plain_kernel_u11(nj, nv, wl);
    }
    return nullptr;
}

// Weights of one chunk in LDS: when they take at most 32 KiB.
bool weights_in_lds(int taps, int NJ, bool tail)
{
    return !tuning().conv_no_wl && (size_t)taps * (NJ * 64 + (tail ? conv::kTailPacked : 0)) * 4 <= 32 * 1024;
}

struct TileChoice {
    bool ok;
    int NJ, jgroups, NV;
    int Tz, Ty, Tx, HZ, HY, HX, MS;
    int cz, cy, cx;
    bool wl, dbuf;
    bool tail;          // NJ full tiles and an 8-map block (direct_mfma_tail_impl.h)
    int cps, splits;    // input-map chunks per workgroup and number of such shares
    size_t lds;
    double cost;        // expected clocks of the launch
};

constexpr int kCUs = 256;
constexpr size_t kConvLdsMax = 64 * 1024;

// A layer with few output voxels leaves most compute units without a workgroup (and the rest
// with one wave per SIMD): below one workgroup per unit the input-map chunks are split over
// gridDim.z until about three per unit exist; the shares' partial sums are added in a fixed
// order afterwards.
void split_chunks(long blocks, int nchunk, int& cps, int& splits)
{
    long want = tuning().conv_no_split || blocks >= kCUs ? 1 : (3 * kCUs + blocks - 1) / blocks;
    if (want > nchunk) want = nchunk;
    cps = (int)(nchunk / want);        // rounded down: shares of equal length, a few more of them
    splits = (nchunk + cps - 1) / cps;
}

// Picks the tile box and the per-wave tile count so that the launch fills the
// 256 compute units in as few, as full rounds as possible.
TileChoice search_tile(int fM, int fK, int dz, int dy, int dx, int kz, int ky, int kx, int spz, int spy, int spx, bool tail)
{
    TileChoice best = {};
    best.ok = false;
    const int taps = kz * ky * kx;
    if (taps > kMaxTaps) return best;
    const int tiles = (fM + 15) / 16;
    const int jgroups = tail ? 1 : (tiles + 7) / 8;
    const int NJ = tail ? fM / 16 : (tiles + jgroups - 1) / jgroups;
    double best_cost = 1e300;
    const int nchunk = (fK + 3) / 4;
    // tuning aid: ZNN_CONV_TILE="NV,Tz,Ty,Tx" pins the configuration
    const int (&pin)[4] = tuning().conv_tile;
    const int nvs[6] = {2, 4, 5, 6, 7, 8};
    for (int ni = 0; ni < 6; ++ni) {
        const int NV = nvs[ni];
        if (tail ? !conv::tail_instance(NJ, NV) : !conv::plain_instance(NJ, NV)) continue;
        if (pin[0] && NV != pin[0]) continue;
        const int cap = 64 * NV;
        for (int Tx = 1; Tx <= dx && Tx <= cap; ++Tx) {
            for (int Ty = 1; Ty <= dy && Tx * Ty <= cap; ++Ty) {
                int Tz = cap / (Tx * Ty);
                if (Tz > dz) Tz = dz;
                if (Tz < 1) continue;
                if (pin[0]) {
                    if (Tx != pin[3] || Ty != pin[2] || pin[1] * Ty * Tx > cap) continue;
                    Tz = pin[1];
                }
                const int HZ = Tz + spz * (kz - 1), HY = Ty + spy * (ky - 1), HX = Tx + spx * (kx - 1);
                long hvol = (long)HZ * HY * HX;
                long MS = hvol;
                MS = (MS + 15) & ~15L;      // whole 64-word spans of 16 voxels x 4 maps
                const bool wl = weights_in_lds(taps, NJ, tail);
                // halo buffers (two that take turns if they fit, else one), the loader's table (one
                // map's box, padded to the workgroup size), the chunk's weights
                const long MSP = (MS + 255) & ~255L;
                const size_t wbytes = wl ? (size_t)taps * (NJ * 64 + (tail ? conv::kTailPacked : 0)) * 4 : 0;
                bool dbuf = true;
                size_t lds = (size_t)(8 * MS + MSP) * 4 + wbytes;
                if (lds > kConvLdsMax) { dbuf = false; lds = (size_t)(4 * MS + MSP) * 4 + wbytes; }
                if (lds > kConvLdsMax) continue;
                const int cz = (dz + Tz - 1) / Tz, cy = (dy + Ty - 1) / Ty, cx = (dx + Tx - 1) / Tx;
                const long blocks = (long)cz * cy * cx * jgroups;
                // shares of the input maps along gridDim.z when the output gives few workgroups (see below)
                int cps, splits;
                split_chunks(blocks, nchunk, cps, splits);
                // time ~ workgroups per compute unit (they share its matrix cores whether they run side
                // by side or one after the other) x (fixed cost of a workgroup + its chunks x (MFMA work +
                // halo fetch)); a unit with a single workgroup has one wave per SIMD and nothing to overlap
                // its waits with (measured on the 2D benchmark layer: 1.4x)
                const long groups = blocks * splits;
                const double rounds = (double)((groups + kCUs - 1) / kCUs) * (groups <= kCUs ? 1.4 : 1.0);
                // an 8-map block costs four short MFMAs per two voxel tiles (about 10 cycles each)
                const double mfma = (double)taps * (NJ * NV * 32.0 + (tail ? ((NV + 1) / 2) * 40.0 : 0.0));
                // halo fetch per chunk: hidden behind the taps with two buffers, else one exposed memory latency
                const double stage = dbuf ? 300.0 + (double)hvol * 4.0 / 256.0 * 2.0 : 1500.0 + (double)hvol * 4.0 / 256.0 * 6.0;
                const double fixed = 3000.0 + (double)MS / 256.0 * 300.0;      // launch, table, zero fill, epilogue
                // among boxes of equal cost the one that is longest along x: longer contiguous runs in the
                // epilogue's stores and in the halo fetch (config 2: 12x6x6 -> 6x6x12, 2 % faster)
                const double cost = rounds * (fixed + cps * (mfma + stage)) - 0.01 * Tx;
                if (cost < best_cost) {
                    best_cost = cost;
                    best.ok = true;
                    best.NJ = NJ; best.jgroups = jgroups; best.NV = NV;
                    best.Tz = Tz; best.Ty = Ty; best.Tx = Tx;
                    best.HZ = HZ; best.HY = HY; best.HX = HX; best.MS = (int)MS;
                    best.cz = cz; best.cy = cy; best.cx = cx;
                    best.wl = wl;
                    best.dbuf = dbuf;
                    best.tail = tail;
                    best.cps = cps; best.splits = splits;
                    best.lds = lds;
                    best.cost = cost;
                }
            }
        }
    }
    return best;
}

// The search walks thousands of candidate boxes (a fraction of a millisecond on the host),
// and every call of a pass asks for the same answer up to three times: remembered per shape.
TileChoice choose_tile(int fM, int fK, int dz, int dy, int dx, int kz, int ky, int kx, int spz, int spy, int spx, long svol)
{
    struct Entry { int key[12]; TileChoice choice; };
    static std::mutex lock;
    static std::vector<Entry> memo;
    const bool tail = tail_applies(fM, svol);
    const int key[12] = {fM, fK, dz, dy, dx, kz, ky, kx, spz, spy, spx, tail ? 1 : 0};
    {
        std::lock_guard<std::mutex> hold(lock);
        for (const Entry& e : memo)
            if (memcmp(e.key, key, sizeof(key)) == 0) return e.choice;
    }
    Entry e;
    memcpy(e.key, key, sizeof(key));
    e.choice = search_tile(fM, fK, dz, dy, dx, kz, ky, kx, spz, spy, spx, tail);
    if (tail && !e.choice.ok) e.choice = search_tile(fM, fK, dz, dy, dx, kz, ky, kx, spz, spy, spx, false);
    std::lock_guard<std::mutex> hold(lock);
    if (memo.size() >= 256) memo.erase(memo.begin());
    memo.push_back(e);
    return e.choice;
}

size_t partial_bytes(const TileChoice& c, int fM, long dvol)
{
    return c.splits > 1 ? align256((size_t)c.splits * fM * dvol * sizeof(float)) : 0;
}

size_t packed_bytes(const TileChoice& c, int fK, int taps)
{
    const size_t per_tap = (size_t)c.NJ * 64 + (c.tail ? conv::kTailPacked : 0);
    return align256((size_t)c.jgroups * ((fK + 3) / 4) * taps * per_tap * sizeof(float));
}

TileChoice choose_for(const Geom& g, bool backward)
{
    return backward ? choose_tile(g.f, g.fo, g.nz, g.ny, g.nx, g.kz, g.ky, g.kx, g.spz, g.spy, g.spx, g.ovol())
                    : choose_tile(g.fo, g.f, g.oz, g.oy, g.ox, g.kz, g.ky, g.kx, g.spz, g.spy, g.spx, g.nvol());
}

}  // namespace

// The tiled path takes every shape whose halo box fits LDS; otherwise the caller falls back.
bool mfma_conv_supported(const Geom& g, bool backward)
{
    const long svol = backward ? g.ovol() : g.nvol();
    if (svol < (1L << 28) && choose_split(g, backward).ok) return true;
    const TileChoice c = choose_for(g, backward);
    // the halo loader addresses the chunk's four source maps with one 32-bit byte offset
    return c.ok && svol < (1L << 28);
}

// Expected seconds of the pass: the search's clocks, the sum of the shares, weight packing.
double mfma_conv_seconds(const Geom& g, bool backward)
{
    if (const SplitChoice p = choose_split(g, backward); p.ok) return p.cost / 1.9e9 + 2e-6;
    const TileChoice c = choose_for(g, backward);
    if (!c.ok) return 2.0 * g.f * g.fo * (double)g.ovol() * g.kvol() / 1e12;
    const double count = backward ? (double)g.f * g.nvol() : (double)g.fo * g.ovol();
    return c.cost / 2.1e9 + (c.splits > 1 ? 4e-6 + 4.0 * count * (c.splits + 1) / 3e12 : 0.0);
}

size_t mfma_conv_workspace(const Geom& g, bool backward)
{
    if (const SplitChoice p = choose_split(g, backward); p.ok)
        return split_packed_bytes(p) +
               (p.splits > 1 ? align256((size_t)p.splits * (backward ? g.f * g.nvol() : g.fo * g.ovol()) * sizeof(float)) : 0);
    const TileChoice c = choose_for(g, backward);
    if (!c.ok) return 0;
    return packed_bytes(c, backward ? g.fo : g.f, (int)g.kvol()) +
           partial_bytes(c, backward ? g.f : g.fo, backward ? g.nvol() : g.ovol());
}

// The pass on packed weights.  With more than one share of the input maps (mfma_conv_splits) the sums go to `partial`, one
// array of result maps per share, and the caller adds them in ascending order.
int mfma_conv_packed(const Geom& g, bool backward, const float* src, const float* wp, float* dst, float* partial,
                     const Finish& finish, hipStream_t s)
{
    if (choose_split(g, backward).ok) return split_conv(g, backward, src, wp, dst, partial, finish, s);
    ConvTile P = {};
    P.src = src; P.dst = dst;
    P.kz = g.kz; P.ky = g.ky; P.kx = g.kx;
    P.spz = g.spz; P.spy = g.spy; P.spx = g.spx;
    if (!backward) {
        P.fK = g.f; P.fM = g.fo;
        P.sz = g.nz; P.sy = g.ny; P.sx = g.nx;
        P.pz = P.py = P.px = 0;
        P.dz = g.oz; P.dy = g.oy; P.dx = g.ox;
    } else {
        P.fK = g.fo; P.fM = g.f;
        P.sz = g.oz; P.sy = g.oy; P.sx = g.ox;
        P.pz = g.spz * (g.kz - 1); P.py = g.spy * (g.ky - 1); P.px = g.spx * (g.kx - 1);
        P.dz = g.nz; P.dy = g.ny; P.dx = g.nx;
    }
    const TileChoice c = choose_for(g, backward);
    if (!c.ok) return fail(ZNN_EUNSUPPORTED, "no tile configuration fits this shape");
    P.Tz = c.Tz; P.Ty = c.Ty; P.Tx = c.Tx;
    P.HZ = c.HZ; P.HY = c.HY; P.HX = c.HX; P.MS = c.MS;
    P.dHX = make_fastdiv((unsigned)c.HX); P.dHY = make_fastdiv((unsigned)c.HY); P.dHZ = make_fastdiv((unsigned)c.HZ);
    P.cz = c.cz; P.cy = c.cy; P.cx = c.cx;
    P.nchunk = (P.fK + 3) / 4;
    P.cps = c.cps;
    P.dbuf = c.dbuf ? 1 : 0;
    if (log_enabled())
        fprintf(stderr, "[znn] conv mfma (%s): NJ=%d%s jgroups=%d NV=%d U=%d tile=%dx%dx%d halo=%dx%dx%d blocks=%d splits=%d lds=%zu buffers=%d\n",
                backward ? "bwd" : "fwd", c.NJ, c.tail ? "+8" : "", c.jgroups, c.NV, group_width(g.kx, g.spx), c.Tz, c.Ty, c.Tx, c.HZ, c.HY, c.HX,
                c.cz * c.cy * c.cx, c.splits, c.lds, c.dbuf ? 2 : 1);
    P.wp = wp;
    P.partial = partial;
    P.y = finish.y; P.bias = finish.bias; P.deriv = finish.deriv;
    const int U = group_width(g.kx, g.spx);
    ConvFn fn = c.tail ? pick_tail_kernel(U, c.NJ, c.NV, c.wl) : pick_plain_kernel(U, c.NJ, c.NV, c.wl);
    if (!fn) return fail(ZNN_EUNSUPPORTED, "no kernel instance for tile %dx%d", c.NJ, c.NV);
    const long blocks = (long)c.cz * c.cy * c.cx;
    if (blocks >= 2147483647L) return fail(ZNN_EUNSUPPORTED, "too many tiles for one launch");
    ZNN_LAUNCH(backward ? "direct backward (MFMA)" : "direct forward (MFMA)", s, fn,
               dim3((unsigned)blocks, (unsigned)c.jgroups, (unsigned)c.splits), dim3(256), c.lds, P);
    return check_launch(backward ? "direct backward (MFMA)" : "direct forward (MFMA)");
}

PackItem mfma_conv_pack_item(const Geom& g, bool backward, const float* w, float* wp)
{
    PackItem p = {};
    p.w = w; p.wp = wp;
    p.f = g.f; p.fo = g.fo;
    p.kz = g.kz; p.ky = g.ky; p.kx = g.kx;
    p.backward = backward ? 1 : 0;
    if (const SplitChoice c = choose_split(g, backward); c.ok) {
        p.split = 1;
        p.NJ = c.NJ; p.nchunk = c.nchunk;
        p.total = (long)c.jgroups * c.nchunk * c.steps * c.NJ * 64;
        return p;
    }
    const TileChoice c = choose_for(g, backward);
    p.NJ = c.NJ; p.nchunk = ((backward ? g.fo : g.f) + 3) / 4;
    p.tail = c.tail ? 1 : 0;
    p.total = (long)c.jgroups * p.nchunk * g.kvol() * (c.NJ * 64 + (c.tail ? conv::kTailPacked : 0));
    return p;
}

template <int N>
static void pack_launch(const PackItem* items, int n, hipStream_t s)
{
    PackArgs<N> A = {};
    unsigned blocks = 0;
    for (; A.n < n; ++A.n) {
        A.item[A.n] = items[A.n];
        A.first[A.n] = blocks;
        blocks += (unsigned)((items[A.n].total + 255) / 256);
    }
    ZNN_LAUNCH("weight packing", s, k_pack_weights<N>, dim3(blocks), dim3(256), 0, A);
}

int mfma_pack_weights(const PackItem* items, int n, hipStream_t s)
{
    if (n == 1) pack_launch<1>(items, 1, s);
    else
        for (int i0 = 0; i0 < n; i0 += kPackItems) pack_launch<kPackItems>(items + i0, std::min(kPackItems, n - i0), s);
    return check_launch("weight packing");
}

size_t mfma_conv_packed_bytes(const Geom& g, bool backward)
{
    if (const SplitChoice p = choose_split(g, backward); p.ok) return split_packed_bytes(p);
    const TileChoice c = choose_for(g, backward);
    return c.ok ? packed_bytes(c, backward ? g.fo : g.f, (int)g.kvol()) : 0;
}

int mfma_conv_splits(const Geom& g, bool backward)
{
    const SplitChoice p = choose_split(g, backward);
    return p.ok ? p.splits : choose_for(g, backward).splits;
}

int mfma_conv(const Geom& g, bool backward, const float* src, const float* w, float* dst, void* ws,
              hipStream_t s)
{
    const PackItem p = mfma_conv_pack_item(g, backward, w, (float*)ws);
    float* partial = (float*)((char*)ws + mfma_conv_packed_bytes(g, backward));
    int rc = mfma_pack_weights(&p, 1, s);
    if (rc == ZNN_OK) rc = mfma_conv_packed(g, backward, src, p.wp, dst, partial, Finish{}, s);
    if (rc != ZNN_OK || mfma_conv_splits(g, backward) == 1) return rc;
    return mfma_conv_sum(g, backward, partial, dst, s);
}

int mfma_conv_sum(const Geom& g, bool backward, const float* partial, float* dst, hipStream_t s)
{
    const long count = backward ? (long)g.f * g.nvol() : (long)g.fo * g.ovol();
    ZNN_LAUNCH("sum over input-map shares", s, k_conv_reduce, dim3((unsigned)((count + 255) / 256)), dim3(256), 0,
               partial, dst, count, mfma_conv_splits(g, backward));
    return check_launch("sum over input-map shares");
}

}  // namespace znn
