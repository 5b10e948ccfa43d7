// Host side of the split direct kernel (direct_split_impl.h): packing of the weights, search for the workgroup's box, launch.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <vector>

#include "direct.h"
#include "direct_beside_impl.h"

namespace znn {

namespace {

using split::BesideTile;
using split::SplitFn;
using split::SplitTile;

// Weights for the split kernel: a thread makes the three parts of eight input maps' weights at one tap, [group][chunk][step]
// [16-map tile][part][lane], negative in every second step.
__device__ __forceinline__ void pack_split(const PackItem& P, long t)
{
    const int taps = P.taps, steps = (taps + split::kTaps - 1) / split::kTaps;
    const int lane = (int)(t & 63);
    unsigned r = (unsigned)(t >> 6);        // a wave's 3 KiB: 2^32 of them are more than any memory
    const int jt = (int)(r % (unsigned)P.NJ); r /= (unsigned)P.NJ;
    const int s = (int)(r % (unsigned)steps); r /= (unsigned)steps;
    const int ic = (int)(r % (unsigned)P.nchunk), jg = (int)(r / (unsigned)P.nchunk);
    const int m = (jg * P.NJ + jt) * 16 + (lane & 15), tap = s * split::kTaps + (lane >> 4);
    const int fM = P.backward ? P.f : P.fo, fK = P.backward ? P.fo : P.f;
    float v[8];
    const float scale = split::step_negative(s, steps, ic) ? -split::kScale : split::kScale;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int k = ic * split::kMaps + e;
        const bool in = m < fM && k < fK && tap < taps;
        const long at = P.backward ? ((long)k * P.f + m) * taps + (taps - 1 - tap) : ((long)m * P.f + k) * taps + tap;
        const float x = P.w[in ? at : 0];       // all eight loads are in flight together
        v[e] = in ? x * scale : 0.f;
    }
    split::uintx4* out = reinterpret_cast<split::uintx4*>(P.wp) + (t >> 6) * 3 * 64 + lane;
#pragma unroll
    for (int p = 0; p < 3; ++p) out[p * 64] = split::take_part8(v);
}

// Several layers and passes at a time: the weights of a round take one launch instead of one per convolution.  N = 1 serves the
// calls of a single layer, whose launch then carries 80 bytes of arguments instead of 2 KB.
constexpr int kPackItems = 24;
template <int N> struct PackArgs { PackItem item[N]; unsigned first[N]; int n; };

template <int N>
__global__ void __launch_bounds__(256) k_pack_weights(PackArgs<N> A)
{
    int q = 0;
    if (N > 1) while (q + 1 < A.n && blockIdx.x >= A.first[q + 1]) ++q;        // uniform
    const long t = (long)(blockIdx.x - A.first[q]) * 256 + threadIdx.x;
    if (t < A.item[q].total) pack_split(A.item[q], t);
}

constexpr int kCUs = 256;
constexpr size_t kLds = 160 * 1024;
constexpr int kMaxTaps = 4096;

// Instances: accumulators (NJ NV tiles) and two sets of weights (24 NJ registers) fit the 256 registers of two waves per SIMD (5 x 2
// tiles all but two of them).
constexpr bool instance(int nj, int nv) { return nj >= 1 && nj <= 5 && nj * nv <= (nj <= 2 ? 16 : nj == 3 ? 18 : nj == 4 ? 12 : 10); }

template <int NJ, int NV, int NW> SplitFn instance_of()
{
    if constexpr (instance(NJ, NV)) return split::k_conv_split<NJ, NV, NW>;
    else return nullptr;
}

template <int NJ, int NW> SplitFn pick_nv(int nv)
{
    switch (nv) {
        case 1: return instance_of<NJ, 1, NW>();
        case 2: return instance_of<NJ, 2, NW>();
        case 3: return instance_of<NJ, 3, NW>();
        case 4: return instance_of<NJ, 4, NW>();
        case 6: return instance_of<NJ, 6, NW>();
        case 8: return instance_of<NJ, 8, NW>();
    }
    return nullptr;
}

template <int NW> SplitFn pick_nj(int nj, int nv)
{
    switch (nj) {
        case 1: return pick_nv<1, NW>(nv);
        case 2: return pick_nv<2, NW>(nv);
        case 3: return pick_nv<3, NW>(nv);
        case 4: return pick_nv<4, NW>(nv);
        case 5: return pick_nv<5, NW>(nv);
    }
    return nullptr;
}

SplitFn pick(int nj, int nv, int nw) { return nw == 8 ? pick_nj<8>(nj, nv) : pick_nj<4>(nj, nv); }

// One axis of a pass: source and result extents, taps, their spacing and the taps of zeros in front.
struct Axis { int s, d, k, sp, p, phases, e; };     // e: longest sublattice of the result
struct Pass { Axis a[3]; int fM, fK; };

Pass pass_of(const Geom& g, bool backward)
{
    Pass P;
    const int n[3] = {g.nz, g.ny, g.nx}, o[3] = {g.oz, g.oy, g.ox}, k[3] = {g.kz, g.ky, g.kx}, sp[3] = {g.spz, g.spy, g.spx};
    for (int d = 0; d < 3; ++d) {
        Axis& a = P.a[d];
        a.s = backward ? o[d] : n[d];
        a.d = backward ? n[d] : o[d];
        a.k = k[d];
        a.sp = k[d] > 1 ? sp[d] : 1;
        a.p = backward ? k[d] - 1 : 0;
        a.phases = std::min(a.sp, a.d);
        a.e = (a.d + a.sp - 1) / a.sp;
    }
    P.fM = backward ? g.f : g.fo;
    P.fK = backward ? g.fo : g.f;
    return P;
}

// Expected clocks of a launch of `groups` workgroups and of the sum of its shares.  Waves that stage in between: fitted to the times of 900 boxes on 22 layers (standard
// deviation 15 %).
struct ClocksBetween {
    int NW, most, fit;
    double step, stage, fixed;
    // of a choice's tiles and waves
    explicit ClocksBetween(const SplitChoice& c) : NW(c.NW)
    {
        // clocks of a step of the workgroup: matrix cores, LDS reads (128 bytes a clock), weights from the vector cache (64)
        step = 0.92 * std::max({c.NW / 4 * c.NJ * c.NV * 96.0, c.NW * c.NV * 24.0, c.NW * c.NJ * 48.0}) + 82.0 * c.NW / 4;
        most = (c.NJ <= 2 && c.NJ * c.NV <= 8 ? 12 : 8) / c.NW;         // workgroups whose registers fit a compute unit
        fixed = 5200.0 + 11.5 * 16 * c.NV * c.NW * c.NJ;
        step *= c.steps;
    }
    // of its halo box
    void set_halo(int hvol, int spx) { stage = 4.0 * hvol * (1.0 + 0.06 * (spx - 1)); }
    void set_lds(size_t lds) { fit = std::max(1, std::min(most, (int)(kLds / lds))); }
    // no number of shares takes less: all chunks of all workgroups of one share, on units that are never idle
    double least(long groups, int nchunk) const { return (1 - 1e-9) * groups / kCUs * nchunk * (step + 0.46 * stage); }
    double operator()(int cps, int splits, long groups, double count) const
    {
        const long per_cu = (groups + kCUs - 1) / kCUs;
        // a unit with one wave per SIMD has nothing to overlap its waits with, one workgroup nothing for its stages
        const long both = std::min((long)fit, per_cu);
        const double alone = both * NW < 8 ? 1.38 : 1.0;
        double cost = per_cu * (fixed + cps * (step * alone + stage * (both > 1 ? 0.46 : 1.0)));
        if (splits > 1) cost += 7000.0 + count * (splits + 1) * 4.0 / 3.0e12 * 2.1e9;
        return cost;
    }
};

int least_groups(int tiles) { return (tiles + 4) / 5; }      // of 16-map tiles

// The larger of two times, and a little more where they are near each other: neither overlaps the other perfectly.
double larger(double a, double b)
{
    const double p = a * a, q = b * b;
    return std::sqrt(std::sqrt(p * p + q * q));
}

// Waves that stage beside: fitted to 5200 choices on 90 layers (standard deviation 12 %).
double clocks_beside(const SplitChoice& c, long groups, int spx, double count)
{
    const int regs = 39 + 41 * c.NJ;
    const int fit = std::max(1, std::min((int)(512 / ((regs + 7) / 8 * 8) * 4 / (split::kBesideWaves + split::kStagers)), (int)(kLds / c.lds)));
    const long per_cu = (groups + kCUs - 1) / kCUs, both = std::min<long>(fit, per_cu);
    const double rounds = (double)groups / kCUs / both;
    // a step: matrix cores, LDS reads, six products of a tile one behind another
    const double busy = larger(c.NJ * 70.7 + 50, (1 + c.NJ) * 55.2), step = larger(busy, 6 * larger(16 * c.NJ, 12.3) + 50);
    const double stage = 1500 + 4.37 * c.H[0] * c.H[1] * c.H[2] * (1 + 0.164 * std::min(3, spx - 1));
    const double ends = 207 + 115 * c.NJ;
    const double one = ends + stage + c.cps * larger(c.steps * step + 600.0, stage);
    const double all = both * (c.cps * c.steps * busy + 6.25 * ends);
    double cost = std::max(1.0, rounds + 0.92 * (std::ceil(rounds) - rounds)) * larger(one, all);
    if (c.splits > 1) cost += 4040.0 + count * (c.splits + 1) * 4.0 / 3.0e12 * 1.3e9;
    // What the least of many is too low by (it is picked for the fit's errors as well), and a tenth more: of those better by less, every tenth was slower.
    return 1.28 * cost * std::pow(c.splits, 0.115) * std::pow(c.NJ, 0.09);
}

// Where waves that stage beside pay: one 16-voxel tile a wave, and one workgroup on a unit or two; with more of them a unit has other workgroups to go on with while one
// stages, and twice the waves that multiply.  An XCD's units take the workgroups of its run of boxes, so those of the longest run count: 81 boxes of three groups, 243 for
// 256 units, are 33 for 32 units, one of which took two after another (12 -> 88 maps, 135 x 26, 5^2: 13.1 us, in between 11.1; by 76 boxes 8.8).
// A thread has four voxels in flight: larger halo boxes take more than one time of memory.
// More groups of the `tiles` of maps than have to be stage a box as often, shares have little to stage ahead: both take short chunks.  And three or four steps a chunk have
// nothing to hide a stage behind, where it is done more often; nor has a single chunk of two or three (1.00 of the time, two tiles of maps 1.01).  Past these lines, by
// the price: three tiles of maps 0.90 of the time between (to 1.20), two voxel tiles 0.91 (to 1.12), three or four shares 0.94, five 0.97.  Groups of two tiles of maps
// with a workgroup on a unit 0.79 on average; with two 1.00 (to 1.03) where a tile is empty, 1.01 (to 1.11) where a second chunk takes the LDS of the other, else 0.92.
bool worth_beside(const SplitChoice& c, long boxes, int tiles)
{
    constexpr int units = kCUs / 8;
    const long groups = (boxes + 7) / 8 * c.jgroups * c.splits;     // of an XCD
    const bool more = c.jgroups > least_groups(tiles), brief = c.steps <= 8, lean = groups <= units && !more;
    const bool two = c.NJ * c.jgroups <= 3 || (tiles == 4 && c.cps == 1);
    return c.H[0] * c.H[1] * c.H[2] <= 4 * 64 * split::kStagers && groups <= (two ? 2 : 1) * units &&
           (!more || (brief && c.jgroups <= 3 && c.splits == 1)) && (c.splits == 1 || (brief && c.splits == 2)) &&
           c.steps > (!lean ? 4 : c.cps == 1 ? 3 : 1);
}

// The best choice of one kind against that of the other.  Where waves in between take shares, the prices are too far off: the sum of few results takes less than its part of
// the price, and one share walks all chunks one after another.  Time beside / between of 1200 passes of drawn layers that the price alone takes beside: no shares between 0.89
// (1.03 at most); shares, up to 40 000 results 1.00 (to 1.18), up to 100 000 0.95 (to 1.11), above 0.80 (to 0.98), five or six tiles of maps 0.97 (to 1.25).
// Of 725 more that the price takes, which neither it nor these lines nor those of worth_beside were fitted to, they leave 670: 0.887 of the time, four above 1.02 (1.08 at most).
bool take_beside(const SplitChoice& beside, const SplitChoice& between, double count)
{
    if (!beside.ok || !between.ok) return beside.ok;
    return beside.cost < between.cost && (between.splits == 1 || (count >= 1e5 && beside.NJ * beside.jgroups <= 4));
}

// the tiles that k_conv_beside has
bool beside_tiles(int nj, int nv, int nw) { return nj <= 2 && nv == 1 && nw == split::kBesideWaves; }

// Beside, a workgroup's LDS: staging buffers and weights (two where there is a chunk to stage behind another), tables.  False: not of this choice.
bool place_beside(SplitChoice& c)
{
    const size_t hvol = (size_t)c.H[0] * c.H[1] * c.H[2], box = hvol * split::kVoxelBytes, weights = (size_t)c.steps * c.NJ * 3 * 1024;
    const int buffers = c.cps > 1 ? 2 : 1;
    c.hop = buffers > 1 ? (int)box : 0;
    c.whop = buffers > 1 ? (int)weights : 0;
    c.wofs = (int)(buffers * box);
    c.tables = (int)(buffers * (box + weights));
    c.lds = c.tables + hvol * 4 + (size_t)(c.steps + 2) * split::kTaps * 4;
    c.beside = beside_tiles(c.NJ, c.NV, c.NW) && c.lds <= kLds;
    return c.beside;
}

bool place_between(SplitChoice& c)
{
    const size_t hvol = (size_t)c.H[0] * c.H[1] * c.H[2];
    c.beside = false;
    c.lds = hvol * (split::kVoxelBytes + 4) + (size_t)(c.steps + 2) * split::kTaps * 4;
    return c.lds <= kLds;
}

// The box of output voxels of a choice, and what follows from it.  Boxes in all, 0: no LDS for the halo box, or too many for the kernels' divisions.
inline long set_box(SplitChoice& c, const Pass& P, int Tz, int Ty, int Tx, int cx)
{
    const int Hz = Tz + P.a[0].k - 1, Hy = Ty + P.a[1].k - 1, Hx = Tx + P.a[2].k - 1;
    if ((size_t)Hz * Hy * Hx * (split::kVoxelBytes + 4) > kLds) return 0;
    const int cz = (P.a[0].e + Tz - 1) / Tz, cy = (P.a[1].e + Ty - 1) / Ty;
    const long boxes = (long)cz * cy * cx * c.phases;
    if ((double)boxes * std::max({c.phases, cx, cy}) >= 4294967296.0) return 0;
    c.T[0] = Tz; c.T[1] = Ty; c.T[2] = Tx;
    c.H[0] = Hz; c.H[1] = Hy; c.H[2] = Hx;
    c.c[0] = cz; c.c[1] = cy; c.c[2] = cx;
    return boxes;
}

// Expected clocks of the launch (and of the sum of its shares) for every box that fits, the least taken.  Waves that stage in between take all maps of as few
// groups as there can be; for waves that stage beside, which have one shape of tiles, more groups are looked at too, where worth_beside can hold at all.  A first call of
// a shape waits for this: 152 us on average over 12000 passes of drawn layers (400 when every tile shape of every number of groups was walked).
SplitChoice search(const Pass& P)
{
    SplitChoice between = {}, other = {};       // the best whose waves stage in between, and beside
    const Axis &az = P.a[0], &ay = P.a[1], &ax = P.a[2];
    const int taps = az.k * ay.k * ax.k;
    if (taps > kMaxTaps) return between;
    SplitChoice c = {};
    c.steps = (taps + split::kTaps - 1) / split::kTaps;
    c.nchunk = (P.fK + split::kMaps - 1) / split::kMaps;
    c.phases = az.phases * ay.phases * ax.phases;
    const int tiles = (P.fM + 15) / 16;
    const double count = (double)P.fM * az.d * ay.d * ax.d;
    const int nvs[6] = {1, 2, 3, 4, 6, 8}, nws[2] = {4, 8};
    const int (&pin)[4] = tuning().conv_tile;
    // a launch has at least so many boxes of one tile for each of the waves that multiply
    const long beside_boxes = c.phases * (((long)az.e * ay.e * ax.e + 16 * split::kBesideWaves - 1) / (16 * split::kBesideWaves));
    int boxes = 0;
    for (int most_nj = 5; most_nj >= 1; --most_nj) {
        c.jgroups = (tiles + most_nj - 1) / most_nj;
        c.NJ = (tiles + c.jgroups - 1) / c.jgroups;
        if (c.NJ != most_nj) continue;
        const bool more = c.jgroups > least_groups(tiles);
        SplitChoice easiest = c;            // for worth_beside
        easiest.splits = 1;
        easiest.cps = c.nchunk;
        for (int d = 0; d < 3; ++d) easiest.H[d] = P.a[d].k;
        const bool may_beside = beside_tiles(c.NJ, 1, split::kBesideWaves) && worth_beside(easiest, beside_boxes, tiles);
        if (more && !may_beside) continue;
        for (int NW : nws)
            for (int NV : nvs) {
                const bool beside = may_beside && beside_tiles(c.NJ, NV, NW);
                if (!instance(c.NJ, NV) || (more && !beside) || (pin[0] && NV * NW != pin[0])) continue;
                c.NV = NV; c.NW = NW;
                const int cap = 16 * NV * NW;
                ClocksBetween clocks_between(c);
                for (int Tx = 1; Tx <= ax.e && Tx <= cap; ++Tx) {
                    const int column = cap / Tx, cx = (ax.e + Tx - 1) / Tx;
                    for (int Ty = 1; Ty <= ay.e && Ty <= column; ++Ty) {
                        if (pin[0] && (Tx != pin[3] || Ty != pin[2] || pin[1] * Ty * Tx > cap)) continue;
                        ++boxes;
                        const long blocks = set_box(c, P, pin[0] ? pin[1] : az.e > 1 ? std::min(column / Ty, az.e) : 1, Ty, Tx, cx);
                        if (!blocks) continue;
                        // extents that a smaller one would replace without another box
                        auto loose = [&](int d) { return c.T[d] > 1 && (P.a[d].e + c.T[d] - 2) / (c.T[d] - 1) == c.c[d]; };
                        const bool stages = beside && (pin[0] || (!loose(2) && !loose(1)));
                        clocks_between.set_halo(c.H[0] * c.H[1] * c.H[2], ax.sp);
                        // most boxes are beyond the best one whatever their shares
                        const bool fits = !more && (!between.ok || clocks_between.least(blocks * c.jgroups, c.nchunk) - 0.01 * Tx <= between.cost) && place_between(c);
                        if (fits) clocks_between.set_lds(c.lds);
                        else if (!stages) continue;
                        for (int splits = 1, cps = c.nchunk; ; ) {
                            const long groups = blocks * c.jgroups * splits;
                            c.splits = splits; c.cps = cps;
                            if (fits) {
                                c.cost = clocks_between(cps, splits, groups, count) - 0.01 * Tx;
                                if (!between.ok || c.cost < between.cost) {
                                    place_between(c);
                                    between = c;
                                    between.ok = true;
                                }
                            }
                            if (stages && worth_beside(c, blocks, tiles) && place_beside(c)) {
                                c.cost = clocks_beside(c, groups, ax.sp, count) - 0.01 * Tx;
                                if (!other.ok || c.cost < other.cost) {
                                    other = c;
                                    other.ok = true;
                                }
                            }
                            // the next smaller share of the chunks, while the chip is not full; of more groups there are none
                            if (more || cps == 1 || groups >= 3 * kCUs || tuning().conv_no_split) break;
                            do ++splits; while ((c.nchunk + splits - 1) / splits == cps);
                            cps = (c.nchunk + splits - 1) / splits;
                            splits = (c.nchunk + cps - 1) / cps;
                        }
                    }
                }
            }
    }
    SplitChoice best = take_beside(other, between, count) ? other : between;
    best.between = between.cost;
    best.boxes = boxes;
    return best;
}

SplitTile split_args(const Geom& g, const SplitChoice& c, const Pass& p, long total, bool backward, const float* src, const float* w, const void* wp, float* dst,
                     float* partial, const Finish& finish, int share0)
{
    SplitTile P = {};
    P.src = src; P.wp = (const split::uintx4*)wp; P.dst = dst;
    P.w = w; P.wm = backward ? g.kvol() : g.f * g.kvol(); P.wk = backward ? g.f * g.kvol() : g.kvol(); P.reflected = backward ? 1 : 0;
    P.fK = p.fK; P.fM = p.fM;
    P.sz = p.a[0].s; P.sy = p.a[1].s; P.sx = p.a[2].s;
    P.pz = p.a[0].p; P.py = p.a[1].p; P.px = p.a[2].p;
    P.dz = p.a[0].d; P.dy = p.a[1].d; P.dx = p.a[2].d;
    P.kz = p.a[0].k; P.ky = p.a[1].k; P.kx = p.a[2].k;
    P.spz = p.a[0].sp; P.spy = p.a[1].sp; P.spx = p.a[2].sp;
    P.Tz = c.T[0]; P.Ty = c.T[1]; P.Tx = c.T[2];
    P.HZ = c.H[0]; P.HY = c.H[1]; P.HX = c.H[2]; P.hvol = c.H[0] * c.H[1] * c.H[2];
    P.cy = c.c[1]; P.cx = c.c[2];
    P.qy = p.a[1].phases; P.qx = p.a[2].phases; P.phases = c.phases;
    P.total = (int)total; P.run = (int)((total + 7) / 8);
    P.nchunk = c.nchunk; P.cps = c.cps; P.steps = c.steps;
    P.share0 = share0;
    P.partial = partial;
    P.y = finish.y; P.bias = finish.bias; P.deriv = finish.deriv;
    P.dHX = make_fastdiv((unsigned)c.H[2]); P.dHY = make_fastdiv((unsigned)c.H[1]);
    P.dTX = make_fastdiv((unsigned)c.T[2]); P.dTY = make_fastdiv((unsigned)c.T[1]);
    P.dKX = make_fastdiv((unsigned)P.kx); P.dKY = make_fastdiv((unsigned)P.ky);
    P.dPH = make_fastdiv((unsigned)P.phases); P.dQX = make_fastdiv((unsigned)P.qx); P.dQY = make_fastdiv((unsigned)P.qy);
    P.dCX = make_fastdiv((unsigned)P.cx); P.dCY = make_fastdiv((unsigned)P.cy);
    return P;
}

BesideTile beside_args(const Geom& g, const SplitChoice& c, const Pass& p, long total, bool backward, const float* src, const float* w, const void* wp, float* dst,
                       float* partial, const Finish& finish, int share0, int shares)
{
    using split::make_boxdiv;
    BesideTile P = {};
    P.total = (int)total; P.run = (int)((total + 7) / 8);
    P.phases = c.phases; P.qx = p.a[2].phases; P.qy = p.a[1].phases;
    P.cx = c.c[2]; P.cy = c.c[1];
    P.dPH = make_boxdiv((unsigned)P.phases); P.dQX = make_boxdiv((unsigned)P.qx); P.dQY = make_boxdiv((unsigned)P.qy);
    P.dCX = make_boxdiv((unsigned)P.cx); P.dCY = make_boxdiv((unsigned)P.cy);
    P.Tz = c.T[0]; P.Ty = c.T[1]; P.Tx = c.T[2];
    P.spz = p.a[0].sp; P.spy = p.a[1].sp; P.spx = p.a[2].sp;
    P.nchunk = c.nchunk; P.cps = c.cps; P.share0 = share0;
    P.hop = c.hop; P.wofs = c.wofs; P.whop = c.whop; P.tables = c.tables;
    P.sz = p.a[0].s; P.sy = p.a[1].s; P.sx = p.a[2].s;
    P.pz = p.a[0].p; P.py = p.a[1].p; P.px = p.a[2].p;
    P.HX = c.H[2]; P.HY = c.H[1]; P.hvol = c.H[0] * c.H[1] * c.H[2];
    P.dHX = make_boxdiv((unsigned)c.H[2]); P.dHY = make_boxdiv((unsigned)c.H[1]);
    P.fK = p.fK; P.src = src; P.wp = (const split::uintx4*)wp;
    P.steps = c.steps;
    P.kz = p.a[0].k; P.ky = p.a[1].k; P.kx = p.a[2].k;
    P.dKX = make_boxdiv((unsigned)P.kx); P.dKY = make_boxdiv((unsigned)P.ky);
    P.dTX = make_boxdiv((unsigned)c.T[2]); P.dTY = make_boxdiv((unsigned)c.T[1]);
    P.fM = p.fM;
    P.dz = p.a[0].d; P.dy = p.a[1].d; P.dx = p.a[2].d;
    P.dst = shares > 1 ? partial : dst;
    P.share = shares > 1 ? (long)P.fM * P.dz * P.dy * P.dx : 0;
    P.y = finish.y; P.bias = finish.bias; P.deriv = finish.deriv;
    P.w = w; P.wm = backward ? g.kvol() : g.f * g.kvol(); P.wk = backward ? g.f * g.kvol() : g.kvol(); P.reflected = backward ? 1 : 0;
    return P;
}

}  // namespace

// The search walks thousands of boxes, and every call of a pass asks several times: remembered per shape.
SplitChoice choose_split(const Geom& g, bool backward)
{
    struct Entry { int key[12]; SplitChoice choice; };
    static std::mutex lock;
    static std::vector<Entry> memo;
    Entry e;
    const int key[12] = {g.f, g.fo, g.nz, g.ny, g.nx, g.kz, g.ky, g.kx, g.spz, g.spy, g.spx, backward ? 1 : 0};
    memcpy(e.key, key, sizeof(key));
    {
        std::lock_guard<std::mutex> hold(lock);
        for (const Entry& m : memo)
            if (memcmp(m.key, key, sizeof(key)) == 0) return m.choice;
    }
    const Pass P = pass_of(g, backward);
    e.choice = SplitChoice{};
    // a lane's byte offset in a source map has 32 bits
    if ((backward ? g.ovol() : g.nvol()) < (1L << 28)) e.choice = search(P);
    std::lock_guard<std::mutex> hold(lock);
    if (memo.size() >= 256) memo.erase(memo.begin());
    memo.push_back(e);
    return e.choice;
}

// A choice whose tiles of maps or chunks of a share are other ones than the search's: staged as before if that can be.  False: no LDS for it.
bool split_place(SplitChoice& c)
{
    return (c.beside && place_beside(c)) || place_between(c);
}

double split_seconds(double clocks) { return clocks / 1.9e9 + 2e-6; }

// Packed weights; one step of padding behind them, which the kernel fetches ahead.
size_t split_packed_bytes(const SplitChoice& c)
{
    return align256(((size_t)c.jgroups * c.nchunk * c.steps + 1) * c.NJ * 3 * 64 * 16);
}

PackItem split_pack_item(const Geom& g, const SplitChoice& c, bool backward, const float* w, void* wp)
{
    PackItem p = {};
    p.w = w; p.wp = wp;
    p.f = g.f; p.fo = g.fo;
    p.taps = (int)g.kvol();
    p.backward = backward ? 1 : 0;
    p.NJ = c.NJ; p.nchunk = c.nchunk;
    p.total = (long)c.jgroups * c.nchunk * c.steps * c.NJ * 64;
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

int split_pack_weights(const PackItem* items, int n, hipStream_t s)
{
    if (n == 1) pack_launch<1>(items, 1, s);
    else
        for (int i0 = 0; i0 < n; i0 += kPackItems) pack_launch<kPackItems>(items + i0, std::min(kPackItems, n - i0), s);
    return check_launch("weight packing");
}

int split_conv(const Geom& g, const SplitChoice& c, bool backward, const float* src, const float* w, const void* wp, float* dst, float* partial,
               const Finish& finish, hipStream_t s, int share0, int shares)
{
    const Pass p = pass_of(g, backward);
    const long total = (long)c.c[0] * c.c[1] * c.c[2] * c.phases;
    if (total >= 2147483640L) return fail(ZNN_EUNSUPPORTED, "too many tiles for one launch");
    if (!shares) shares = c.splits;
    if (log_enabled())
        fprintf(stderr, "[znn] conv split (%s): NJ=%d jgroups=%d NV=%d waves=%d tile=%dx%dx%d halo=%dx%dx%d blocks=%ld splits=%d-%d/%d %s lds=%zu cost=%.0f of %d boxes\n",
                backward ? "bwd" : "fwd", c.NJ, c.jgroups, c.NV, c.NW, c.T[0], c.T[1], c.T[2], c.H[0], c.H[1], c.H[2], total, share0,
                share0 + shares, c.splits, c.beside ? "beside" : "between", c.lds, c.cost, c.boxes);
    const char* const name = backward ? "direct backward (MFMA)" : "direct forward (MFMA)";
    const dim3 grid((unsigned)(total + 7) / 8 * 8, (unsigned)c.jgroups, (unsigned)shares);
    if (c.beside) {
        ZNN_LAUNCH(name, s, c.NJ == 1 ? split::k_conv_beside<1> : split::k_conv_beside<2>, grid, dim3(64 * (split::kBesideWaves + split::kStagers)), c.lds,
                   beside_args(g, c, p, total, backward, src, w, wp, dst, partial, finish, share0, shares));
    } else {
        const SplitFn fn = pick(c.NJ, c.NV, c.NW);
        if (!fn) return fail(ZNN_EUNSUPPORTED, "no kernel instance for tile %dx%d", c.NJ, c.NV);
        ZNN_LAUNCH(name, s, fn, grid, dim3(64 * c.NW), c.lds, split_args(g, c, p, total, backward, src, w, wp, dst, partial, finish, share0));
    }
    return check_launch(name);
}

}  // namespace znn
