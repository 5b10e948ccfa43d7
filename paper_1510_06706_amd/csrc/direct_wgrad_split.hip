// Host side of the split kernel gradient (direct_wgrad_split_impl.h): the copies of the images, the search for the shape of
// the launch, the launch and the sum of the shares.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <vector>

#include "direct.h"
#include "direct_wgrad_split_impl.h"

namespace znn {

namespace {

using namespace split;

// One image in vectors: on every axis, vector (r - r0) V + q - q0 holds voxels r + (e Q + q) sp of the pieces e < E (r: residue modulo
// the tap spacing sp); vectors q from `real` on, and voxels outside the image, are zero.
struct SplitImage {
    const float* src; uintx4* dst;
    int n[3], sp[3], real[3], V[3], all[3], r0[3], q0[3];      // all: vectors of all residues
    int step[3], log2E[3];  // Q sp, E
    long vectors;
    int signs;              // 1: steps (four vectors along x) change their sign along every axis
    unsigned first;         // workgroup it starts at
    FastDiv dvol, dall[3], dV[3];   // product of all, all, V
};
constexpr int kGradJobs = 8;        // layers that share a launch of k_split_images
struct SplitArgs { SplitImage image[2 * kGradJobs]; int n; };

// A thread makes one vector: eight loads (neighbouring lanes along x), the split, three 16-byte stores.  Bound by memory.
__global__ void __launch_bounds__(256) k_split_images(SplitArgs A)
{
    int q = 0;
    while (q + 1 < A.n && blockIdx.x >= A.image[q + 1].first) ++q;      // uniform
    const SplitImage& S = A.image[q];
    const long t = (long)(blockIdx.x - S.first) * 256 + threadIdx.x;
    if (t >= S.vectors) return;
    const unsigned vol = S.dvol.d;
    const unsigned map = S.vectors < 2147483648L ? fdiv_any((unsigned)t, S.dvol) : (unsigned)(t / vol);
    const unsigned r = (unsigned)(t - (long)map * vol);
    // an axis may be long: quotients have to be exact for any dividend
    const unsigned row = fdiv_any(r, S.dall[2]), vx = r - row * S.all[2], vz = fdiv_any(row, S.dall[1]), vy = row - vz * S.all[1];
    const int hx = (int)fdiv_any(vx, S.dV[2]), hy = (int)fdiv_any(vy, S.dV[1]), hz = (int)fdiv_any(vz, S.dV[0]);
    const int rx = S.r0[2] + hx, ry = S.r0[1] + hy, rz = S.r0[0] + hz;
    const int x = S.q0[2] + (int)vx - hx * S.V[2], y = S.q0[1] + (int)vy - hy * S.V[1], z = S.q0[0] + (int)vz - hz * S.V[0];
    const float* src = S.src + map * ((long)S.n[0] * S.n[1] * S.n[2]);
    const bool real = (z < S.real[0]) & (y < S.real[1]) & (x < S.real[2]);
    const float scale = S.signs && ((vx / 4 + vy + vz) & 1) ? -kScale : kScale;
    const int z0 = rz + z * S.sp[0], y0 = ry + y * S.sp[1], x0 = rx + x * S.sp[2];
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        // e as (e_z, e_y, e_x)
        const int ex = e & ((1 << S.log2E[2]) - 1), ey = e >> S.log2E[2] & ((1 << S.log2E[1]) - 1), ez = e >> (S.log2E[2] + S.log2E[1]);
        const int gz = z0 + ez * S.step[0], gy = y0 + ey * S.step[1], gx = x0 + ex * S.step[2];
        const bool in = real & (gz < S.n[0]) & (gy < S.n[1]) & (gx < S.n[2]);
        unsigned at = (gz * S.n[1] + gy) * S.n[2] + gx;     // a map has less than 2^30 voxels
        asm volatile("" : "+v"(at));        // not a branch around it, which would wait for the load before
        const float w = src[in ? at : 0u];
        v[e] = in ? w * scale : 0.f;
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) S.dst[t * 3 + p] = take_part8(v);
}

// The sums over the shares in ascending order.  Threads run along the columns of the partial sums, which are read once per share;
// gw[j][i][tap] of a column is written wherever it lies.
struct GradSumArgs { const float* partial; float* gw; WgradSum S; long slots; };
__global__ void __launch_bounds__(256) k_wgrad_sum(GradSumArgs A)
{
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    long from, to;
    if (t >= A.slots || !wgrad_slot(A.S, t, from, to)) return;
    const long step = (long)A.S.planes * A.S.Mpad * A.S.Npad;
    float acc = 0.f;
#pragma unroll 4
    for (int s = 0; s < A.S.ksplit; ++s) acc += A.partial[s * step + from];
    A.gw[to] = acc;
}

// The same for small layers with many shares, where one thread per element is a long chain of additions on few threads: wave l
// sums the shares l, l + 4, ... of 64 elements, then the four sums are added in order.
__global__ void __launch_bounds__(256) k_wgrad_sum4(GradSumArgs A)
{
    __shared__ float part[4][64];
    const int l = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long t = (long)blockIdx.x * 64 + lane;
    long from, to;
    const bool live = t < A.slots && wgrad_slot(A.S, t, from, to);
    const long step = (long)A.S.planes * A.S.Mpad * A.S.Npad;
    float acc = 0.f;
    if (live) {
#pragma unroll 4
        for (int s = l; s < A.S.ksplit; s += 4) acc += A.partial[s * step + from];
    }
    part[l][lane] = acc;
    __syncthreads();
    if (l == 0 && live) A.gw[to] = ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
}

// Instances: NJ NT accumulators, the operands of a step and the sums of two column tiles in the 256 registers of two waves per SIMD.
constexpr bool instance(int nj, int nt) { return nj >= 1 && nj <= 5 && nt >= 1 && nt <= 8 && nj * nt <= (nj <= 3 ? 24 : 20); }

template <int NJ, int NT> GradFn instance_of()
{
    if constexpr (instance(NJ, NT)) return k_wgrad_split<NJ, NT>;
    else return nullptr;
}

template <int NJ> GradFn pick_nt(int nt)
{
    switch (nt) {
        case 1: return instance_of<NJ, 1>();
        case 2: return instance_of<NJ, 2>();
        case 3: return instance_of<NJ, 3>();
        case 4: return instance_of<NJ, 4>();
        case 5: return instance_of<NJ, 5>();
        case 6: return instance_of<NJ, 6>();
        case 7: return instance_of<NJ, 7>();
        case 8: return instance_of<NJ, 8>();
    }
    return nullptr;
}

GradFn pick(int nj, int nt)
{
    switch (nj) {
        case 1: return pick_nt<1>(nt);
        case 2: return pick_nt<2>(nt);
        case 3: return pick_nt<3>(nt);
        case 4: return pick_nt<4>(nt);
        case 5: return pick_nt<5>(nt);
    }
    return nullptr;
}

struct GradChoice {
    bool ok;
    int E[3], Q[3], R[3], H[3], P[3], I[3], T[3], ph[3];
    int GA, GB, planes_a, planes_b, NJ, JG, NT, KW, G, GS, IS, tiles, tps, shares;
    double cost;            // expected clocks
};

constexpr int kCUs = 256;

// bytes of a map in LDS, 16 more per `mod`-residue wanted: `units` 16-byte units rounded up to `want` modulo 16
int pitch(int units, int want)
{
    while (units % 16 != want % 16) ++units;
    return units * 16;
}

// Shapes of a launch, priced in clocks of the shader: the steps of the busiest wave (six MFMAs of 16 clocks per product, two waves
// per SIMD), the copies of the tiles, what a step, a tile and a workgroup cost besides, the copies of the images and the sum of the
// shares.  Constants fitted to the times of 1100 shapes on 25 layers (standard deviation 10 %).
GradChoice search(const Geom& g)
{
    GradChoice best = {};
    const int o[3] = {g.oz, g.oy, g.ox}, k[3] = {g.kz, g.ky, g.kx}, spacing[3] = {g.spz, g.spy, g.spx};
    int sp[3], ph[3], u[3];         // tap spacing, residues that hold voxels, voxels of the longest residue
    for (int d = 0; d < 3; ++d) {
        sp[d] = k[d] > 1 ? spacing[d] : 1;
        ph[d] = std::min(sp[d], o[d]);
        u[d] = (o[d] + sp[d] - 1) / sp[d];
    }
    const int phases = ph[0] * ph[1] * ph[2];
    const int mt = (g.fo + 15) / 16;
    for (int ez = 1; ez <= 8; ez *= 2)
        for (int ey = 1; ez * ey <= 8; ey *= 2) {
            const int E[3] = {ez, ey, 8 / (ez * ey)};
            int Q[3];
            bool fits = true;
            for (int d = 0; d < 3; ++d) {
                Q[d] = (u[d] + E[d] - 1) / E[d];
                fits = fits && (E[d] == 1 || (E[d] - 1) * Q[d] < u[d]);     // no piece without a voxel
            }
            // small layers may have no such cut: then the longest axis, and pieces of zeros
            if (!fits && !(E[0] == 1 && E[1] == 1)) continue;
            for (int ga = 1; ga <= k[0]; ga = ga < k[0] && 2 * ga > k[0] ? k[0] : 2 * ga)
                for (int gb = 1; gb <= k[1]; gb = gb < k[1] && 2 * gb > k[1] ? k[1] : 2 * gb) {
                    if (ga > 1 && gb < k[1]) continue;
                    const int planes_a = (k[0] + ga - 1) / ga, planes_b = (k[1] + gb - 1) / gb, planes = planes_a * planes_b;
                    const int tg = ga * gb * k[2], ncols = g.f * tg, ct = (ncols + 15) / 16;
                    for (int JG = (mt + 4) / 5; JG <= (mt + 4) / 5 + 1 && JG <= mt; ++JG) {
                        const int NJ = (mt + JG - 1) / JG;
                        for (int KW = 1; KW <= 8; KW *= 2)
                            for (int NT = 1; NT <= 8; ++NT) {
                                if (!instance(NJ, NT)) break;
                                const int NG = kGradWaves / KW;
                                const int G = (ct + NG * NT - 1) / (NG * NT);
                                if (NT > 1 && (ct + NG * (NT - 1) - 1) / (NG * (NT - 1)) == G) continue;      // fewer would do
                                const int cols = NT * NG * 16;
                                const long other = (long)planes * G * JG;
                                const double step = 1.52 * 192.0 * NJ * NT, fixed = 12600.0 + 460.0 * NJ * NT;
                                if ((double)g.f * tg * tg >= 4294967296.0) continue;    // fdiv of column numbers
                                // the matrix instructions alone, evenly spread over the chip
                                if (best.ok && (double)Q[0] * Q[1] * ((Q[2] + 3) / 4) * phases / KW * step * other / kCUs + fixed >= best.cost) continue;
                                const int maps = std::min(g.f, G == 1 ? g.f : (cols + tg - 2) / tg + 1);
                                for (int X = 4; X <= (Q[2] + 3) / 4 * 4 && X <= 64; X += 4) {
                                    const int tx = (Q[2] + X - 1) / X;
                                    if (X > 4 && (Q[2] + X - 5) / (X - 4) == tx) continue;    // a shorter tile gives as many
                                    for (int Ry = 1; Ry <= Q[1] && Ry <= 8; ++Ry)
                                        for (int Rz = 1; Rz <= Q[0] && Rz <= (Ry == Q[1] ? 8 : 1); ++Rz) {
                                            const int R[3] = {Rz, Ry, X}, H[3] = {Rz + ga - 1, Ry + gb - 1, X + k[2] - 1};
                                            const int gu = Rz * Ry * X * 3, iu = H[0] * H[1] * H[2] * 3;
                                            // sixteen rows of an operand on different banks: maps an odd number of 16-byte units
                                            // apart (gout); columns, taps along x first, evenly spaced (in)
                                            const int GS = pitch(gu, gu | 1), IS = pitch(iu, 3 * k[2]);
                                            const long bytes = (long)NJ * 16 * GS + (long)maps * IS;
                                            const long real = (long)std::min(g.fo, NJ * 16) * GS + (long)maps * IS;
                                            if (bytes > kGradBuffer) break;
                                            if ((std::min(g.fo, NJ * 16) * GS + 1023) / 1024 + ((long)maps * IS + 1023) / 1024 > kGradSpans * kGradWaves) break;
                                            const int steps = Rz * Ry * X / 4, wsteps = (steps + KW - 1) / KW;
                                            const long T[3] = {(Q[0] + Rz - 1) / Rz, (Q[1] + Ry - 1) / Ry, tx};
                                            const long tiles = T[0] * T[1] * T[2] * phases;
                                            const double tile = std::max(wsteps * (step + 230.0), real / 18.5 + 230.0 * wsteps) + 580.0;
                                            for (int rounds = 1; rounds <= 4; ++rounds) {
                                                long shares = std::max(1L, (long)kCUs * rounds / other);
                                                if (rounds > 1 && other > kCUs * (rounds - 1L)) continue;
                                                shares = std::min(shares, tiles);
                                                const long tps = (tiles + shares - 1) / shares;
                                                shares = (tiles + tps - 1) / tps;
                                                const long run = (shares * other + 7) / 8;
                                                const double sums = (double)shares * planes * g.fo * ct * 16 * 4.0;
                                                double V = 0;
                                                {
                                                    double a = g.fo, b = g.f;
                                                    for (int d = 0; d < 3; ++d) { a *= (double)ph[d] * T[d] * R[d]; b *= (double)ph[d] * (T[d] * R[d] + k[d] - 1); }
                                                    V = a + b;
                                                }
                                                const double cost = std::ceil(run / 32.0) * (tps * tile + fixed) + sums / 4.5e12 * 2.1e9 + V * 80.0 / 5.0e12 * 2.1e9;
                                                if (best.ok && cost >= best.cost) continue;
                                                best.ok = true;
                                                best.cost = cost;
                                                for (int d = 0; d < 3; ++d) {
                                                    best.E[d] = E[d]; best.Q[d] = Q[d]; best.R[d] = R[d]; best.H[d] = H[d];
                                                    best.T[d] = (int)T[d];
                                                    best.ph[d] = ph[d];
                                                    best.P[d] = ph[d] * (int)T[d] * R[d]; best.I[d] = best.P[d] + ph[d] * (k[d] - 1);
                                                }
                                                best.GA = ga; best.GB = gb; best.planes_a = planes_a; best.planes_b = planes_b;
                                                best.NJ = NJ; best.JG = JG; best.NT = NT; best.KW = KW; best.G = G;
                                                best.GS = GS; best.IS = IS;
                                                best.tiles = (int)tiles; best.tps = (int)tps; best.shares = (int)shares;
                                            }
                                        }
                                }
                            }
                    }
                }
        }
    return best;
}

size_t vectors(const int (&v)[3], int maps) { return (size_t)maps * v[0] * v[1] * v[2]; }

// The images are copied, and the gradient summed, in slabs along the first axis that has tiles to share out, so that the copies of
// large layers take 128 MiB and not several times the images (a slab is a few launches; below that size one is best: two slabs of
// 40 + 40 maps of 64^3 voxels cost 2 % more than one of 112 MB).
constexpr size_t kCopies = (size_t)128 << 20;
struct Slabs { int axis, residues, rows; size_t bytes; };       // residues and tile rows of a residue in a slab, bytes of its copies

Slabs slabs_of(const Geom& g, const GradChoice& c)
{
    const int k[3] = {g.kz, g.ky, g.kx};
    Slabs S = {};
    S.axis = c.ph[0] * c.T[0] > 1 ? 0 : 1;
    const int d = S.axis;
    auto bytes = [&](int residues, int rows) {
        int p[3], i[3];
        for (int a = 0; a < 3; ++a) { p[a] = c.P[a]; i[a] = c.I[a]; }
        p[d] = residues * rows * c.R[d];
        i[d] = residues * (rows * c.R[d] + k[d] - 1);
        return align256(vectors(p, g.fo) * kVectorBytes) + align256(vectors(i, g.f) * kVectorBytes);
    };
    S.residues = c.ph[d]; S.rows = c.T[d];
    if (bytes(S.residues, S.rows) > kCopies) {
        S.residues = 1;
        const int slabs = (int)std::min((size_t)c.T[d], (bytes(1, S.rows) + kCopies - 1) / kCopies);
        S.rows = (c.T[d] + slabs - 1) / slabs;
        while (S.rows > 1 && bytes(1, S.rows) > kCopies) --S.rows;
    }
    S.bytes = bytes(S.residues, S.rows);
    return S;
}

// The kernels index voxels of a map and 16-byte units of a slab's copies with 32 bits.
bool indexes_fit(const Geom& g, const GradChoice& c)
{
    return g.nvol() < (1L << 30) && slabs_of(g, c).bytes / kPartBytes < (1L << 31);
}

GradChoice choose(const Geom& g)
{
    struct Entry { int key[14]; GradChoice choice; };
    static std::mutex lock;
    static std::vector<Entry> memo;
    Entry e;
    const int key[14] = {g.f, g.fo, g.nz, g.ny, g.nx, g.kz, g.ky, g.kx, g.spz, g.spy, g.spx, g.oz, g.oy, g.ox};
    memcpy(e.key, key, sizeof(key));
    {
        std::lock_guard<std::mutex> hold(lock);
        for (const Entry& m : memo)
            if (memcmp(m.key, key, sizeof(key)) == 0) return m.choice;
    }
    e.choice = search(g);
    if (e.choice.ok && !indexes_fit(g, e.choice)) e.choice.ok = false;
    std::lock_guard<std::mutex> hold(lock);
    if (memo.size() >= 256) memo.erase(memo.begin());
    memo.push_back(e);
    return e.choice;
}

}  // namespace

bool split_grad_supported(const Geom& g) { return choose(g).ok; }

double split_grad_seconds(const Geom& g)
{
    const GradChoice c = choose(g);
    if (!c.ok) return 2.0 * g.f * g.fo * (double)g.ovol() * g.kvol() / 1e12;
    return c.cost / 2.1e9 + 8e-6;
}

// columns of the partial sums, whole tiles of them
static size_t columns_of(const Geom& g, const GradChoice& c) { return ((size_t)g.f * c.GA * c.GB * g.kx + 15) / 16 * 16; }

// the partial sums, and the copies of the images that only the pass itself needs
size_t split_grad_sums_bytes(const Geom& g)
{
    const GradChoice c = choose(g);
    if (!c.ok) return 0;
    return align256((size_t)c.shares * c.planes_a * c.planes_b * g.fo * columns_of(g, c) * sizeof(float));
}

size_t split_grad_copies_bytes(const Geom& g)
{
    const GradChoice c = choose(g);
    return c.ok ? slabs_of(g, c).bytes : 0;
}

namespace {

// One slab of a layer's gradient, as its launches take it.
struct GradJob {
    GradTile P;
    SplitImage image[2];
    unsigned copy_blocks[2];
    GradFn fn;
};

int log_grad(const GradChoice& c, const Slabs& slabs)
{
    return fprintf(stderr, "[znn] wgrad split: NJ=%d JG=%d NT=%d G=%d KW=%d pieces=%dx%dx%d tile=%dx%dx%d halo=%dx%dx%d taps=%dx%d planes=%d tiles=%d tps=%d shares=%d slab=%dx%d cost=%.0f\n",
                   c.NJ, c.JG, c.NT, c.G, c.KW, c.E[0], c.E[1], c.E[2], c.R[0], c.R[1], c.R[2], c.H[0], c.H[1], c.H[2], c.GA, c.GB,
                   c.planes_a * c.planes_b, c.tiles, c.tps, c.shares, slabs.residues, slabs.rows, c.cost);
}

// The slab of `residues` residues from r0 and `rows` tile rows from row0 on; tps: tiles of a share (0: set here, by the first slab).
int make_job(const Geom& g, const GradChoice& c, int d0, int r0, int residues, int row0, int rows, const GradItem& item, int& tps, GradJob& job)
{
    const int n[3] = {g.nz, g.ny, g.nx}, o[3] = {g.oz, g.oy, g.ox}, k[3] = {g.kz, g.ky, g.kx}, sp[3] = {g.spz, g.spy, g.spx};
    const int planes = c.planes_a * c.planes_b;
    job.fn = pick(c.NJ, c.NT);
    if (!job.fn) return fail(ZNN_EUNSUPPORTED, "no kernel instance for tile %dx%d", c.NJ, c.NT);
    GradTile& P = job.P;
    P = GradTile{};
    P.in = item.in; P.gout = item.gout; P.partial = item.partial;
    P.f = g.f; P.fo = g.fo;
    P.GA = c.GA; P.GB = c.GB; P.planes_b = c.planes_b; P.planes = planes;
    P.GS = c.GS; P.IS = c.IS;
    P.steps = c.R[0] * c.R[1] * c.R[2] / 4;
    P.KW = c.KW; P.G = c.G; P.JG = c.JG;
    P.Mpad = g.fo; P.Npad = (int)columns_of(g, c);
    P.dX4 = make_fastdiv((unsigned)(c.R[2] / 4)); P.dRX = make_fastdiv((unsigned)c.R[2]); P.dRY = make_fastdiv((unsigned)c.R[1]);
    P.dHX = make_fastdiv((unsigned)c.H[2]); P.dHY = make_fastdiv((unsigned)c.H[1]);
    P.dGU = make_fastdiv((unsigned)c.GS / 16); P.dIU = make_fastdiv((unsigned)c.IS / 16);
    P.dTG = make_fastdiv((unsigned)(c.GA * c.GB * k[2])); P.dKX = make_fastdiv((unsigned)k[2]); P.dGB = make_fastdiv((unsigned)c.GB);
    SplitImage &sg = job.image[0], &si = job.image[1];
    sg = si = SplitImage{};
    sg.src = item.gout; si.src = item.in;
    int ph[3];
    for (int d = 0; d < 3; ++d) {
        const bool cut = d == d0;
        ph[d] = cut ? residues : c.ph[d];
        P.T[d] = cut ? rows : c.T[d];
        P.r0[d] = cut ? r0 : 0; P.q0[d] = cut ? row0 * c.R[d] : 0;
        P.n[d] = n[d]; P.o[d] = o[d]; P.k[d] = k[d]; P.sp[d] = k[d] > 1 ? sp[d] : 1;
        P.E[d] = c.E[d]; P.Q[d] = c.Q[d]; P.R[d] = c.R[d]; P.H[d] = c.H[d];
        P.P[d] = ph[d] * P.T[d] * c.R[d];
        P.I[d] = P.P[d] + ph[d] * (k[d] - 1);
        for (SplitImage& S : job.image) {
            S.step[d] = c.Q[d] * P.sp[d]; S.log2E[d] = c.E[d] / 2 - c.E[d] / 8;     // 0 to 3 of 1, 2, 4, 8
            S.sp[d] = P.sp[d]; S.r0[d] = P.r0[d]; S.q0[d] = P.q0[d];
        }
        sg.n[d] = o[d]; sg.all[d] = P.P[d]; sg.V[d] = P.P[d] / ph[d]; sg.real[d] = c.Q[d];
        si.n[d] = n[d]; si.all[d] = P.I[d]; si.V[d] = P.I[d] / ph[d]; si.real[d] = c.Q[d] + k[d] - 1;
    }
    sg.signs = 1;
    sg.vectors = (long)vectors(P.P, g.fo);
    si.vectors = (long)vectors(P.I, g.f);
    sg.dst = (uintx4*)item.copies;
    si.dst = (uintx4*)((char*)item.copies + align256(vectors(P.P, g.fo) * kVectorBytes));
    P.gs = sg.dst; P.is = si.dst;
    for (SplitImage& S : job.image) {
        for (int d = 0; d < 3; ++d) { S.dall[d] = make_fastdiv((unsigned)S.all[d]); S.dV[d] = make_fastdiv((unsigned)S.V[d]); }
        S.dvol = make_fastdiv((unsigned)S.all[0] * S.all[1] * S.all[2]);
    }
    const long blocks0 = (sg.vectors + 255) / 256, blocks1 = (si.vectors + 255) / 256;
    P.tiles_y = ph[1] * P.T[1]; P.tiles_x = ph[2] * P.T[2];
    P.tiles = ph[0] * P.T[0] * P.tiles_y * P.tiles_x;
    if (!tps) tps = (P.tiles + c.shares - 1) / c.shares;
    P.tps = tps;
    const long total = (long)((P.tiles + tps - 1) / tps) * planes * c.G * c.JG;
    if (blocks0 + blocks1 >= 2147483647L || total >= 2147483640L) return fail(ZNN_EUNSUPPORTED, "too many tiles for one launch");
    job.copy_blocks[0] = (unsigned)blocks0; job.copy_blocks[1] = (unsigned)blocks1;
    P.total = (int)total; P.run = (int)((total + 7) / 8);
    return ZNN_OK;
}

// Copies of all jobs (at most kGradJobs of them) in one launch, then the gradients.
void launch_jobs(const GradJob* jobs, int count, hipStream_t s)
{
    SplitArgs A = {};
    unsigned blocks = 0;
    for (int q = 0; q < count; ++q)
        for (int i = 0; i < 2; ++i) {
            A.image[A.n] = jobs[q].image[i];
            A.image[A.n++].first = blocks;
            blocks += jobs[q].copy_blocks[i];
        }
    ZNN_LAUNCH("split of images", s, k_split_images, dim3(blocks), dim3(256), 0, A);
    for (int q = 0; q < count; ++q)
        ZNN_LAUNCH("direct kernel gradient (MFMA)", s, jobs[q].fn, dim3((unsigned)jobs[q].P.run * 8), dim3(64 * kGradWaves), 0, jobs[q].P);
}

WgradSum shares_of(const Geom& g, const GradChoice& c, const GradJob& first)
{
    WgradSum S = {};
    const int k[3] = {g.kz, g.ky, g.kx};
    S.ksplit = (first.P.tiles + first.P.tps - 1) / first.P.tps; S.planes = first.P.planes; S.planes_b = c.planes_b;
    S.Mpad = first.P.Mpad; S.Npad = first.P.Npad;
    S.f = g.f; S.GA = c.GA; S.GB = c.GB;
    for (int d = 0; d < 3; ++d) S.k[d] = k[d];
    S.columns = g.f * c.GA * c.GB * k[2];
    S.slots = (long)g.fo * S.planes * S.columns;
    S.four = S.slots < 65536 && S.ksplit >= 16 ? 1 : 0;
    return S;
}

}  // namespace

int split_grad(const Geom& g, const GradItem& item, hipStream_t s)
{
    const GradChoice c = choose(g);
    if (!c.ok) return fail(ZNN_EUNSUPPORTED, "no tile configuration fits this shape");
    const Slabs slabs = slabs_of(g, c);
    const int d0 = slabs.axis;
    if (log_enabled()) log_grad(c, slabs);
    GradJob job;
    int tps = 0;            // the first slab is the largest: the others have no more shares than it
    bool more = false;
    for (int r = 0; r < c.ph[d0]; r += slabs.residues)
        for (int row = 0; row < c.T[d0]; row += slabs.rows) {
            const int rc = make_job(g, c, d0, r, slabs.residues, row, std::min(slabs.rows, c.T[d0] - row), item, tps, job);
            if (rc != ZNN_OK) return rc;
            job.P.more = more;
            if (!more) *item.sum = shares_of(g, c, job);
            launch_jobs(&job, 1, s);
            more = true;
        }
    return check_launch("direct kernel gradient (MFMA)");
}

// Copies of at most 8 MiB, three workgroups per compute unit, leave a launch of their own mostly waiting: three layers of the six-layer 3D
// net on a 12^3 patch (40 maps of 24^3, 21^3 and 19^3) took 22 us in three launches; together 305 -> 291 us a round (the line lies
// between two measured rounds).  Two layers
// of 40 maps of 34^3 and 28^3 with sparse taps, 16 MiB and 8 MiB, gained nothing by it: 640 -> 643 us, copies no longer in the cache.
bool split_grad_joins(const Geom& g)
{
    const GradChoice c = choose(g);
    if (!c.ok) return false;
    const Slabs slabs = slabs_of(g, c);
    return slabs.residues == c.ph[slabs.axis] && slabs.rows == c.T[slabs.axis] && slabs.bytes <= (size_t)8 << 20;
}

// Gradients of layers that split_grad_joins takes
int split_grads(const GradItem* items, int count, hipStream_t s)
{
    for (int q0 = 0; q0 < count; q0 += kGradJobs) {
        const int n = std::min(kGradJobs, count - q0);
        GradJob jobs[kGradJobs];
        for (int q = 0; q < n; ++q) {
            const GradItem& item = items[q0 + q];
            const Geom& g = *item.g;
            const GradChoice c = choose(g);
            const Slabs slabs = slabs_of(g, c);
            if (log_enabled()) log_grad(c, slabs);
            int tps = 0;
            const int rc = make_job(g, c, slabs.axis, 0, slabs.residues, 0, slabs.rows, item, tps, jobs[q]);
            if (rc != ZNN_OK) return rc;
            *item.sum = shares_of(g, c, jobs[q]);
        }
        launch_jobs(jobs, n, s);
    }
    return check_launch("direct kernel gradient (MFMA)");
}

int sum_shares(const WgradSum& S, const float* partial, float* gw, hipStream_t s)
{
    GradSumArgs A = {};
    A.S = S; A.partial = partial; A.gw = gw; A.slots = S.slots;
    if (S.four) ZNN_LAUNCH("kernel gradient reduction", s, k_wgrad_sum4, dim3((unsigned)((S.slots + 63) / 64)), dim3(256), 0, A);
    else        ZNN_LAUNCH("kernel gradient reduction", s, k_wgrad_sum, dim3((unsigned)((S.slots + 255) / 256)), dim3(256), 0, A);
    return check_launch("kernel gradient reduction");
}

}  // namespace znn
