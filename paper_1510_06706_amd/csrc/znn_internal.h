// Internal declarations shared by the host-side API and the kernel launchers.
// Nothing in here is part of the public boundary (that is include/znn.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "znn.h"

namespace znn {

// ---------------------------------------------------------------- errors
void set_error(const char* fmt, ...);
int  fail(int code, const char* fmt, ...);
// Checks hipGetLastError() after a launch; returns ZNN_OK or ZNN_EHIP.
int  check_launch(const char* what);

// ---------------------------------------------------------------- kernel-level tracing
// While tracing is on, every launch is bracketed by two HIP events on its stream.
struct TraceScope {
    TraceScope(const char* name, hipStream_t s);
    ~TraceScope();
    int slot;
    hipStream_t stream;
};
#define ZNN_LAUNCH(name, stream, kern, grid, block, lds, ...)                 \
    do {                                                                      \
        znn::TraceScope _ts(name, stream);                                    \
        hipLaunchKernelGGL(kern, grid, block, lds, stream, __VA_ARGS__);      \
    } while (0)

// ---------------------------------------------------------------- geometry
struct Geom {
    int f, fo;            // fan-in, fan-out
    int nz, ny, nx;       // image extents n
    int kz, ky, kx;       // kernel extents k
    int spz, spy, spx;    // sparsity s: neighbouring taps are s voxels apart (Section 2)
    int oz, oy, ox;       // n' = n - s (k - 1)
    int Nz, Ny, Nx, Nxh;  // FFT extents and N_x/2+1
    __host__ __device__ long nvol() const { return (long)nz * ny * nx; }
    __host__ __device__ long kvol() const { return (long)kz * ky * kx; }
    __host__ __device__ long ovol() const { return (long)oz * oy * ox; }
    __host__ __device__ long svol() const { return (long)Nz * Ny * Nxh; }   // complex elements per spectrum
};

inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Smallest 2^a 3^b 5^c >= n.
int  next_fft_extent(int n);
// Largest FFT extent the LDS-resident passes accept.
constexpr int kMaxFftExtent = 1024;

// Division of small unsigned numbers by a launch constant without a hardware divide:
// q = (n * M) >> 32 with M = floor(2^32 / d) + 1 is exact while n * d < 2^32.
struct FastDiv {
    unsigned d, M;
};
inline FastDiv make_fastdiv(unsigned d)
{
    FastDiv f;
    f.d = d;
    f.M = d <= 1 ? 0u : (unsigned)(((1ull << 32) / d) + 1ull);
    return f;
}
__device__ __forceinline__ unsigned fdiv(unsigned n, FastDiv f)
{
    return f.d <= 1 ? n : __umulhi(n, f.M);
}
// The same for any n with n + d < 2^32: n M / 2^32 lies less than one above n / d.
__host__ __device__ __forceinline__ unsigned fdiv_any(unsigned n, FastDiv f)
{
    if (f.d <= 1) return n;
    const unsigned q = (unsigned)((unsigned long)n * f.M >> 32);
    return q * f.d > n ? q - 1 : q;
}

// Tuning aids.  The environment is read exactly once, the first time anything asks (plan
// creation at the latest), and never on a launch path; none of them changes a data layout.
struct Tuning {
    bool log;                   // ZNN_LOG: print launch configurations to stderr
    bool conv_no_split;         // ZNN_CONV_NO_SPLIT: never split the input maps over workgroups
    int  conv_tile[4];          // ZNN_CONV_TILE="T,Tz,Ty,Tx": pin the output box, T 16-voxel tiles (0 = not pinned)
    int  fft_mac_z0;            // ZNN_FFT_MAC_Z0: frequencies per thread of the folded multiply-accumulate / 4
    bool fft_mac_valu;          // ZNN_FFT_MAC_VALU: folded multiply-accumulate on the vector ALUs only
    bool fft_wgrad_plain;       // ZNN_FFT_WGRAD_PLAIN: per-z pruned DFT instead of the radix-4 grouped one
    bool fft_no_fused_xy;       // ZNN_FFT_NO_FUSED_XY: separate x and y passes even where one launch can take both
    bool fft_no_two_level;      // ZNN_FFT_NO_TWO_LEVEL: 256-point strided passes through the LDS radix passes
    bool fft_no_mac_inverse;    // ZNN_FFT_NO_MAC_INVERSE: inverse transform along z as a pass of its own, never inside the multiply-accumulate
    bool fft_no_taps_pass;      // ZNN_FFT_NO_TAPS_PASS: kernels take the general fused x/y pass
    int  fft_lds_kb;            // ZNN_FFT_LDS_KB: LDS per workgroup of the LDS passes (pencils per workgroup follow); 0 = per pass kind
    bool fft_no_tiles;          // ZNN_FFT_NO_TILES: whole-volume transforms where the library would choose tiles
    bool fft_lds_passes;        // ZNN_FFT_LDS_PASSES: LDS passes instead of register passes
};
const Tuning& tuning();
inline bool log_enabled() { return tuning().log; }

// ---------------------------------------------------------------- direct method
int direct_fwd(const Geom& g, const float* in, const float* w, float* out, void* ws, hipStream_t s);
size_t direct_fwd_least(const Geom& g);         // bytes that direct_fwd_groups needs
int direct_fwd_groups(const Geom& g, const float* in, const float* w, float* out, void* ws, hipStream_t s);
int direct_bwd(const Geom& g, const float* gout, const float* w, float* gin, void* ws, hipStream_t s);
int direct_wgrad(const Geom& g, const float* in, const float* gout, float* gw, void* ws, hipStream_t s);
size_t direct_workspace_bytes(const Geom& g, int pass);
// The passes in pieces, for rounds that pack the weights of all layers at once and finish several sums in one launch
struct PackItem { const float* w; void* wp; int f, fo, taps, backward, NJ, nchunk; long total; };
bool conv_takes_packed(const Geom& g, bool backward);       // else it takes the weights as they are
PackItem conv_pack_item(const Geom& g, bool backward, const float* w, void* wp);
int conv_pack_weights(const PackItem* items, int n, hipStream_t s);
size_t conv_packed_bytes(const Geom& g, bool backward);
int conv_splits(const Geom& g, bool backward);
// what a pass does with its finished sums v: y = fn(v + bias[map]) beside v (forward), or v times fn's derivative at the
// forward result `deriv` (backward); the kernels themselves take the rectifier only
struct Finish { float* y; const float* bias; const float* deriv; int fn; };
int conv_pass(const Geom& g, bool backward, const float* src, const float* w, const void* wp, float* dst, float* partial,
              const Finish& finish, hipStream_t s);
int conv_sum(const Geom& g, bool backward, const float* partial, float* dst, hipStream_t s);
size_t grad_sums_bytes(const Geom& g);          // the shares' partial sums
size_t grad_copies_bytes(const Geom& g);        // what the pass itself needs
// Partial sums of a kernel gradient, [share][tap group][Mpad][Npad], and how to add them: in ascending order of the shares
// (k_wgrad_sum), or four interleaved sums per element (k_wgrad_sum4).  Columns of a group are (input map, tap of the group).
struct WgradSum { int ksplit, planes, planes_b, Mpad, Npad, f, GA, GB, k[3], columns, four; long slots; };
int grad_partial(const Geom& g, const float* in, const float* gout, float* partial, void* copies, WgradSum* sum, hipStream_t s);
// The same for several layers that grad_joins takes, whose images are copied by one launch; no two have the same memory for sums or copies.
struct GradItem { const Geom* g; const float* in; const float* gout; float* partial; void* copies; WgradSum* sum; };
bool grad_joins(const Geom& g);
bool grad_is_few(const Geom& g);         // on the vector ALUs
int grads_partial(const GradItem* items, int count, hipStream_t s);
// Element number t of (output map, tap group, column): where a share has it and where the gradient does.  false: a tap
// behind the last one.
__device__ __forceinline__ bool wgrad_slot(const WgradSum& S, long t, long& from, long& to)
{
    unsigned n, plane, j;
    auto place = [&](auto r) {
        n = (unsigned)(r % (unsigned)S.columns); r /= (unsigned)S.columns;
        plane = (unsigned)(r % (unsigned)S.planes);
        j = (unsigned)(r / (unsigned)S.planes);
    };
    if (S.slots <= 4294967295L) place((unsigned)t);         // uniform
    else place((unsigned long)t);
    const unsigned tg = S.GA * S.GB * S.k[2], i = n / tg, q = n - i * tg, c = q % S.k[2], r = q / S.k[2];
    const int b = plane % S.planes_b * S.GB + r % S.GB, a = plane / S.planes_b * S.GA + r / S.GB;
    from = ((long)plane * S.Mpad + j) * S.Npad + n;
    to = ((((long)j * S.f + i) * S.k[0] + a) * S.k[1] + b) * S.k[2] + c;
    return a < S.k[0] && b < S.k[1];
}
// expected seconds of a pass (choice between the methods where nothing has been measured)
double conv_seconds(const Geom& g, bool backward);
double grad_seconds(const Geom& g);

// ---------------------------------------------------------------- FFT method
// Layout of a layer's kernel spectra, fixed when its plan is created (or by
// znn_plan_set_spectra_layout) and carried by the plan from then on, so that the size query,
// the kernel transform and every multiply-accumulate read the same decision.
//   on = false : full spectra [f'][f][N_z][N_y][N_x/2+1] (Section 4, memoized kernel transforms)
//   on = true  : half spectra [f'][f][taps][P], transformed along the fast axes only; the sum
//                over the `taps` planes of the slowest axis (extent N) is taken inside the
//                multiply-accumulate, 4*z0 frequencies per thread
struct Fold { bool on; int N, taps, P, z0; };
Fold fold_full();
// The library's own choice: half spectra where the folded multiply-accumulate applies and the
// layer has enough frequencies to fill the chip, else full spectra.
Fold fold_default(const Geom& g);
// Half spectra whenever the folded multiply-accumulate can take the layer at all (on = false if not).
Fold fold_forced(const Geom& g);

// Tiling of a layer whose FFT passes run on overlapping tiles (fft_tile.hip): transform lengths M, voxels B by
// which tiles advance, T tiles per axis (z, y, x); blocks of 16 frequencies per tile spectrum.
struct Tiling { bool on; int M[3], B[3], T[3]; int tiles, blocks; double seconds; };    // seconds: expected per round

struct FftWorkspace {
    size_t total;
    size_t off_a, off_b;        // spectra of the two node sets of the pass
    size_t off_w;               // kernel spectra (when not resident)
    size_t off_t1, off_t2;      // partially inverted pair volumes (kernel gradient)
};
FftWorkspace fft_workspace(const Geom& g, const Fold& F, int pass, bool resident);
size_t fft_spectra_bytes(const Geom& g, const Fold& F);
int fft_kernel_spectra(const Geom& g, const Fold& F, const float* w, float2* What, hipStream_t s);
int fft_fwd(const Geom& g, const Fold& F, const float* in, const float* w, const float2* resident, float* out,
            void* ws, float2* memo_in, hipStream_t s);
int fft_bwd(const Geom& g, const Fold& F, const float* gout, const float* w, const float2* resident, float* gin,
            void* ws, float2* memo_gout, hipStream_t s);
int fft_wgrad(const Geom& g, const float* in, const float* gout, float* gw, void* ws, hipStream_t s);
int fft_wgrad_from_spectra(const Geom& g, const float2* Ihat, const float2* Ghat, float* gw, void* ws,
                           hipStream_t s);

// Multiply-accumulate with the kernel transform's last axis folded in (fft_mac.hip):
// Wh holds half spectra [pair][tap][P]; X, Y are node spectra [node][N][P].
constexpr int kMaxFoldedTaps = 16;
// z0 = 4, 2 or 1: frequencies per thread along the folded axis are 4 * z0; a thread serves
// fft_mac_group(z0) result nodes.
constexpr int fft_mac_group(int z0) { return z0 == 1 ? 8 : 4; }
int fft_mac_fused(bool backward, int taps, int z0, int f, int fo, int N, int P, const float2* Wh,
                  const float2* X, float2* Y, hipStream_t s);

// The same with the rebuild of the kernel spectrum on the matrix cores (fft_mac_mfma.hip); takes
// extents divisible by 32.
bool fft_mac_mfma_supported(int taps, int N, int P);
bool fft_mac_mfma_can_invert(int taps, int N, int P, int nout);
int fft_mac_mfma(bool backward, int taps, int f, int fo, int N, int P, const float2* Wh, const float2* X,
                 float2* Y, int zinv_o0, int zinv_no, hipStream_t s);
// (zinv_no > 0: the rows [zinv_o0, zinv_o0 + zinv_no) of Y receive the inverse transform of the sums along
// the folded axis instead of the sums; only where fft_mac_mfma_can_invert says so)

// Strided-axis FFT pass with one pencil per thread, whole pencil in registers (fft_reg.hip).
// Pencil (oa, ob, l), l < L, has its element e at in + oa*in_sa + ob*in_sb + l + e*stride;
// elements outside [i0, i0+ni) are taken as zero, only [o0, o0+no) are written.
struct RegAxis {
    const float2* in; float2* out;
    int N, i0, ni, o0, no;
    long stride;
    int L, Oa, Ob;
    long in_sa, in_sb, out_sa, out_sb;
    FastDiv fL;
};
bool fft_axis_reg_supported(int N);
int  fft_axis_reg(RegAxis P, int dir, hipStream_t s);

// Strided-axis FFT passes of lengths N = N1 * N2 above the register limit, N1, N2 <= 16, in two levels with
// the samples in registers at both (fft_two_level.hip).  Pencil (oa, ob, oc, l), l < L, has element e at
// in + oa*in_sa + ob*in_sb + oc*in_sc + l + e*in_stride; elements outside [i0, i0+ni) are taken as zero,
// only [o0, o0+no) are written.
struct TwoLevelAxis {
    const float2* in; float2* out;
    int N, i0, ni, o0, no;
    long in_stride, out_stride;
    int L, Oa, Ob, Oc;
    long in_sa, in_sb, in_sc, out_sa, out_sb, out_sc;
    int chunks;                     // chunks of 16 neighbouring pencils per run of L (filled by the launcher)
    FastDiv fchunks, foc, fob;
};
bool fft_axis_two_level_supported(int N);
int  fft_axis_two_level(TwoLevelAxis P, int dir, hipStream_t s);

// x-axis passes with one row per thread and the row's transform in registers (fft_x_reg*.hip).
// r2c: rows of `sx` real samples (contiguous, `rows` = maps * sz * sy of them) land zero-extended from
// offset ox in lines of N = 2 (Nxh - 1); row (map, z, y) goes to spectrum row (map, z*tz + oz, y*ty + oy).
struct XRegR2C {
    const float* src; float2* dst;
    long rows;
    int sz, sy, sx;
    int Nz, Ny, Nxh;
    int oz, oy, ox;
    int tz, ty;
    FastDiv fsy, fsz;
};
// c2r: spectrum rows (map, z + cz, y + cy), z < dz, y < dy, become contiguous rows of the dx real
// samples from offset cx, times `scale`.
struct XRegC2R {
    const float2* src; float* dst;
    long rows;
    int cz, cy, cx;
    int dz, dy, dx;
    int Nz, Ny, Nxh;
    float scale;
    FastDiv fdy, fdz;
};
// x and y passes in one launch for volumes with equal x and y transform lengths N (fft_xy_reg*.hip):
// a (map, z) plane per workgroup.  forward: planes = maps * sz real planes of sy rows x sx samples, placed
// at (z * tz + oz, oy, ox); inverse: planes = maps * dz spectrum planes z + cz, cropped to rows [cy, cy+dy)
// and samples [cx, cx+dx), times `scale`.
struct XYFwd {
    const float* src; float2* dst;
    long planes;
    int sz, sy, sx;
    int Nz, oz, oy, ox, tz;
};
struct XYInv {
    const float2* src; float* dst;
    long planes;
    int dz, dy, dx;
    int Nz, cz, cy, cx;
    float scale;
};
bool fft_xy_reg_supported(int N);
int  fft_xy_fwd_reg(const XYFwd& P, int N, hipStream_t s);
int  fft_xy_inv_reg(const XYInv& P, int N, hipStream_t s);
bool fft_x_reg_supported(int N);
int  fft_x_r2c_reg(const XRegR2C& P, int N, hipStream_t s);
int  fft_x_c2r_reg(const XRegC2R& P, int N, hipStream_t s);

// ---------------------------------------------------------------- fill (autotuner)
int fill_pattern(float* p, long count, float scale, hipStream_t s);

// max-filter backward, times the derivative of the transfer function that gave y (y may be NULL)
int maxfilter_bwd(int32_t maps, znn_vec3 n, znn_vec3 win, znn_vec3 sp, const float* gout, const int32_t* idx, float* gin,
                  const float* y, int fn, hipStream_t s);
int check_filter(int32_t maps, znn_vec3 n, znn_vec3 win, znn_vec3 sp, bool pool);

// ---------------------------------------------------------------- passes of a plan with buffers given by the caller
size_t plan_pass_bytes(const znn_plan* p, int pass, bool resident);
size_t plan_kernel_bytes(const znn_plan* p);        // spectra of the kernels
size_t plan_memo_bytes(const znn_plan* p);          // spectra of images and gradients
// Kernel spectra of a pass: held by the caller (w NULL), or made from w by the pass itself, at `made` or (NULL) in its workspace.
struct KernelSpectra { const float* w; const float2* held; float2* made; };
// forward: a = in, b = w, result = out; backward: gout, w, gin; kernel gradient: in, gout, gw.  The spectra that b stands for: `resident`, or,
// where that is NULL, made at more->made or in the workspace.
// What a round asks of a pass of the FFT method beside its result: where the kernel spectra go, the kernel gradient beside the backward pass
// (from the node spectra in `memo`, where plan_joins_gradient), and what follows the sums, which the pass does if it can (`finished`).
struct PassMore { float2* made; float* gw; Finish finish; bool finished; };
bool plan_joins_gradient(const znn_plan* p);        // within the workspace that the kernel gradient takes on its own
int plan_pass(const znn_plan* p, int pass, const float* a, const float* b, float* result, const float2* resident, void* ws,
              float2* memo, hipStream_t s, PassMore* more = nullptr);
int plan_wgrad_memo(const znn_plan* p, float2* memo, float* gw, void* ws, hipStream_t s);
// the forward pass in less than its workspace: on tiles in as little as it would take on whole volumes
size_t plan_forward_least(const znn_plan* p);
int plan_forward_within(znn_plan* p, const float* in, const float* w, float* out, void* ws, size_t bytes, hipStream_t s);

}  // namespace znn

struct znn_plan {
    znn_conv_desc desc;
    znn::Geom g;
    int mode;                    // ZNN_DIRECT or ZNN_FFT
    znn::Fold fold;              // layout of this layer's kernel spectra (FFT method)
    znn::Tiling tile;            // overlapping tiles instead of whole volumes (FFT method, layout left to the library)
    const float2* resident;      // kernel spectra held by the caller, or nullptr
    float2* memo;                // caller's buffer for memoized node spectra, or nullptr
    size_t memo_bytes;           // and its size
    bool memo_has_in, memo_has_gout;
    size_t round_memory;         // what a program may hold of this layer beside the workspace of its passes
};
