// Host side of the C ABI: validation, plans, dispatch, autotuner cache.
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <tuple>
#include <vector>

#include "fft_tile.h"

#include <algorithm>

namespace znn {

static thread_local char g_err[512] = "";

void set_error(const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

int fail(int code, const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

int check_launch(const char* what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(ZNN_EHIP, "%s: %s", what, hipGetErrorString(e));
    return ZNN_OK;
}

// ---------------------------------------------------------------- tracing
struct TraceEntry { const char* name; hipEvent_t e0, e1; };
static std::mutex g_trace_mu;
static bool g_trace_on = false;
static std::vector<TraceEntry> g_trace;

TraceScope::TraceScope(const char* name, hipStream_t s) : slot(-1), stream(s)
{
    if (!g_trace_on) return;
    std::lock_guard<std::mutex> lk(g_trace_mu);
    TraceEntry e;
    e.name = name;
    if (hipEventCreate(&e.e0) != hipSuccess) return;
    if (hipEventCreate(&e.e1) != hipSuccess) { (void)hipEventDestroy(e.e0); return; }
    (void)hipEventRecord(e.e0, s);
    g_trace.push_back(e);
    slot = (int)g_trace.size() - 1;
}

TraceScope::~TraceScope()
{
    if (slot < 0) return;
    std::lock_guard<std::mutex> lk(g_trace_mu);
    if (slot < (int)g_trace.size()) (void)hipEventRecord(g_trace[slot].e1, stream);
}

const Tuning& tuning()
{
    static const Tuning t = [] {
        auto flag = [](const char* name) { const char* e = getenv(name); return e && *e && *e != '0'; };
        auto num = [](const char* name, int dflt) { const char* e = getenv(name); return e && *e ? atoi(e) : dflt; };
        Tuning v = {};
        v.log = flag("ZNN_LOG");
        v.conv_no_split = flag("ZNN_CONV_NO_SPLIT");
        if (const char* e = getenv("ZNN_CONV_TILE"))
            if (sscanf(e, "%d,%d,%d,%d", &v.conv_tile[0], &v.conv_tile[1], &v.conv_tile[2], &v.conv_tile[3]) != 4)
                v.conv_tile[0] = v.conv_tile[1] = v.conv_tile[2] = v.conv_tile[3] = 0;
        v.fft_mac_z0 = num("ZNN_FFT_MAC_Z0", 0);
        v.fft_mac_valu = flag("ZNN_FFT_MAC_VALU");
        v.fft_wgrad_plain = flag("ZNN_FFT_WGRAD_PLAIN");
        v.fft_no_taps_pass = flag("ZNN_FFT_NO_TAPS_PASS");
        v.fft_no_two_level = flag("ZNN_FFT_NO_TWO_LEVEL");
        v.fft_no_mac_inverse = flag("ZNN_FFT_NO_MAC_INVERSE");
        v.fft_lds_kb = num("ZNN_FFT_LDS_KB", 0);
        if (v.fft_lds_kb < 8 || v.fft_lds_kb > 64) v.fft_lds_kb = 0;
        v.fft_no_fused_xy = flag("ZNN_FFT_NO_FUSED_XY");
        v.fft_no_tiles = flag("ZNN_FFT_NO_TILES");
        v.fft_lds_passes = flag("ZNN_FFT_LDS_PASSES");
        return v;
    }();
    return t;
}

int next_fft_extent(int n)
{
    for (int m = n;; ++m) {
        int t = m;
        while (t % 2 == 0) t /= 2;
        while (t % 3 == 0) t /= 3;
        while (t % 5 == 0) t /= 5;
        if (t == 1) return m;
    }
}

// ---------------------------------------------------------------- autotune cache
using DescKey = std::tuple<int, int, int, int, int, int, int, int, int, int, int>;
static std::mutex g_tune_mu;
static std::map<DescKey, int> g_tune;

static DescKey key_of(const znn_conv_desc& d)
{
    return DescKey(d.fan_in, d.fan_out, d.image.z, d.image.y, d.image.x, d.kernel.z, d.kernel.y, d.kernel.x,
                   d.sparsity.z, d.sparsity.y, d.sparsity.x);
}

static int validate_desc(const znn_conv_desc* d, Geom* g)
{
    if (!d) return fail(ZNN_EINVAL, "descriptor is NULL");
    if (d->fan_in < 1 || d->fan_out < 1)
        return fail(ZNN_EINVAL, "fan_in and fan_out must be >= 1 (got %d, %d)", d->fan_in, d->fan_out);
    const int n[3] = {d->image.z, d->image.y, d->image.x};
    const int k[3] = {d->kernel.z, d->kernel.y, d->kernel.x};
    const int sp[3] = {d->sparsity.z, d->sparsity.y, d->sparsity.x};
    for (int a = 0; a < 3; ++a) {
        if (n[a] < 1 || k[a] < 1) return fail(ZNN_EINVAL, "image and kernel extents must be >= 1");
        if (sp[a] < 1) return fail(ZNN_EINVAL, "sparsity must be >= 1");
        if ((long)sp[a] * (k[a] - 1) + 1 > n[a])
            return fail(ZNN_EINVAL, "kernel extent %d (sparsity %d) exceeds image extent %d on axis %d",
                        k[a], sp[a], n[a], a);
    }
    if (d->mode != ZNN_DIRECT && d->mode != ZNN_FFT && d->mode != ZNN_AUTO)
        return fail(ZNN_EINVAL, "unknown mode %d", d->mode);
    g->f = d->fan_in; g->fo = d->fan_out;
    g->nz = n[0]; g->ny = n[1]; g->nx = n[2];
    g->kz = k[0]; g->ky = k[1]; g->kx = k[2];
    g->spz = sp[0]; g->spy = sp[1]; g->spx = sp[2];
    g->oz = n[0] - sp[0] * (k[0] - 1); g->oy = n[1] - sp[1] * (k[1] - 1); g->ox = n[2] - sp[2] * (k[2] - 1);
    if ((double)g->nvol() >= 2147483648.0)
        return fail(ZNN_EUNSUPPORTED, "image volume does not fit 32-bit voxel offsets");
    g->Nz = next_fft_extent(n[0]); g->Ny = next_fft_extent(n[1]); g->Nx = next_fft_extent(n[2]);
    g->Nxh = g->Nx / 2 + 1;
    return ZNN_OK;
}

// ---------------------------------------------------------------- FFT method: whole volumes or tiles
// How the library runs a layer by the FFT method when the layout of the kernel spectra is left to it.
struct FftWay { Fold fold; Tiling tile; };

// Seconds of a training round on whole volumes, from the rates of those kernels: 12 ps per spectrum element and forward
// transform, 8.5 ps inverse; per edge and element 0.35 ps per multiply-accumulate with the kernel spectra rebuilt on the matrix
// cores, 0.7 on the vector ALUs, 1.7 streamed in full, and 0.6 for the kernel gradient; 16 launches.
static double whole_volume_seconds(const Geom& g, const Fold& F)
{
    const double sv = (double)g.svol(), nodes = g.f + g.fo, pairs = (double)g.f * g.fo;
    const double mac = !F.on ? 1.7e-12 : fft_mac_mfma_supported(F.taps, F.N, F.P) ? 0.35e-12 : 0.7e-12;
    return sv * (1.5 * nodes * 12e-12 + nodes * 8.5e-12 + pairs * (2.0 * mac + 0.6e-12));
}

static FftWay fft_way(const Geom& g)
{
    FftWay w = {fold_default(g), Tiling{}};
    if (tuning().fft_no_tiles) return w;
    // the spectra live in the buffer that the layout's size query describes
    w.tile = tile_search(g, fft_spectra_bytes(g, w.fold));
    if (!w.tile.on) return w;
    const double whole = whole_volume_seconds(g, w.fold) + 16 * 4e-6, tiles = w.tile.seconds + 11 * 4e-6;
    if (log_enabled())
        fprintf(stderr, "znn: fft %d -> %d of %dx%dx%d: tiles %dx%dx%d, %d of them, %.1f us; whole volumes %.1f us\n", g.f, g.fo,
                g.nz, g.ny, g.nx, w.tile.M[0], w.tile.M[1], w.tile.M[2], w.tile.tiles, tiles * 1e6, whole * 1e6);
    if (whole < tiles) w.tile.on = false;
    return w;
}

// Choice behind mode = auto when no measurement is cached: the expected time of a training round by either method, each
// from the work of the kernels that would run (the searches for their tiles price it) with a factor and a constant.  On 693
// layers of nets of width 6 to 64, timed by znn_autotune, picking by it costs 0.2 % over always picking the faster method.
static int model_choice(const Geom& g)
{
    if (g.Nz > kMaxFftExtent || g.Ny > kMaxFftExtent || g.Nx > kMaxFftExtent) return ZNN_DIRECT;
    const FftWay w = fft_way(g);
    const double fft = w.tile.on ? w.tile.seconds : whole_volume_seconds(g, w.fold);
    const double direct = conv_seconds(g, false) + conv_seconds(g, true) + grad_seconds(g);
    if (log_enabled()) fprintf(stderr, "znn: auto: direct %.1f us, fft %.1f us\n", direct * 1e6, fft * 1e6);
    return 1.2 * fft + 80e-6 < 1.1 * direct + 16e-6 ? ZNN_FFT : ZNN_DIRECT;
}

static size_t fft_pass_bytes(const Geom& g, const FftWay& w, int pass, bool resident)
{
    if (!w.tile.on) return fft_workspace(g, w.fold, pass, resident).total;
    const size_t need = tile_workspace_bytes(g, w.tile, pass, resident);
    // forward and backward: the same workspace serves the plan once it is set to the default layout of whole volumes
    return pass == ZNN_PASS_WGRAD ? std::max(need, align256(sizeof(float2) * (size_t)g.svol()) * (g.f + g.fo))
                                  : std::max(need, fft_workspace(g, w.fold, pass, resident).total);
}

static size_t fft_memo_bytes(const Geom& g, const FftWay& w)
{
    const size_t whole = align256(sizeof(float2) * (size_t)(g.f + g.fo) * g.svol());
    return w.tile.on ? std::max(whole, tile_node_bytes(g, w.tile, g.f) + tile_node_bytes(g, w.tile, g.fo)) : whole;
}

// the half of a memo buffer that holds the spectra of the output gradients
static float2* memo_gradients(const Geom& g, const FftWay& w, float2* memo)
{
    if (!w.tile.on) return memo + (size_t)g.f * g.svol();
    return (float2*)((char*)memo + tile_node_bytes(g, w.tile, g.f));
}

static int run_kernel_spectra(const Geom& g, const FftWay& y, const float* w, float2* What, hipStream_t s)
{
    return y.tile.on ? tile_kernel_spectra(g, y.tile, w, What, s) : fft_kernel_spectra(g, y.fold, w, What, s);
}

// Whole volumes: spectra that do not belong in the workspace are made first.
static int whole_kernels(const Geom& g, const FftWay& y, const KernelSpectra& K, const float2** resident, hipStream_t s)
{
    *resident = K.held ? K.held : K.made;
    return !K.held && K.made ? fft_kernel_spectra(g, y.fold, K.w, K.made, s) : ZNN_OK;
}

static int run_fft_fwd(const Geom& g, const FftWay& y, const float* in, const KernelSpectra& K, float* out,
                       void* ws, float2* memo_in, hipStream_t s, const Finish& finish = {})
{
    if (y.tile.on)
        return tile_fwd(g, y.tile, in, K, out, ws, tile_workspace_bytes(g, y.tile, ZNN_PASS_FWD, K.held || K.made), memo_in, finish, s);
    const float2* resident;
    const int rc = whole_kernels(g, y, K, &resident, s);
    return rc != ZNN_OK ? rc : fft_fwd(g, y.fold, in, K.w, resident, out, ws, memo_in, s);
}

static int run_fft_bwd(const Geom& g, const FftWay& y, const float* gout, const KernelSpectra& K, float* gin,
                       void* ws, float2* memo_gout, hipStream_t s, const Finish& finish = {}, const TileGrad& grad = {})
{
    if (y.tile.on) return tile_bwd(g, y.tile, gout, K, gin, ws, memo_gout, finish, grad, s);
    const float2* resident;
    const int rc = whole_kernels(g, y, K, &resident, s);
    return rc != ZNN_OK ? rc : fft_bwd(g, y.fold, gout, K.w, resident, gin, ws, memo_gout, s);
}

static int run_fft_wgrad(const Geom& g, const FftWay& y, const float* in, const float* gout, float* gw, void* ws, hipStream_t s)
{
    return y.tile.on ? tile_wgrad(g, y.tile, in, gout, gw, ws, s) : fft_wgrad(g, in, gout, gw, ws, s);
}

static int run_fft_wgrad_from_spectra(const Geom& g, const FftWay& y, const float2* Ihat, const float2* Ghat, float* gw,
                                      void* ws, hipStream_t s)
{
    return y.tile.on ? tile_wgrad_from_spectra(g, y.tile, Ihat, Ghat, gw, ws, s)
                     : fft_wgrad_from_spectra(g, Ihat, Ghat, gw, ws, s);
}

static FftWay way_of(const znn_plan* p) { return FftWay{p->fold, p->tile}; }

size_t plan_pass_bytes(const znn_plan* p, int pass, bool resident)
{
    return p->mode == ZNN_DIRECT ? direct_workspace_bytes(p->g, pass) : fft_pass_bytes(p->g, way_of(p), pass, resident);
}

size_t plan_kernel_bytes(const znn_plan* p) { return fft_spectra_bytes(p->g, p->fold); }
size_t plan_memo_bytes(const znn_plan* p) { return fft_memo_bytes(p->g, way_of(p)); }

int plan_pass(const znn_plan* p, int pass, const float* a, const float* b, float* result, const float2* resident, void* ws,
              float2* memo, hipStream_t s, PassMore* more)
{
    const Geom& g = p->g;
    const KernelSpectra K = {resident ? nullptr : b, resident, more ? more->made : nullptr};
    Finish finish = {};
    if (more && (more->finish.y || more->finish.deriv) && p->mode == ZNN_FFT && p->tile.on && more->finish.fn == ZNN_RECTIFY) {
        finish = more->finish;
        more->finished = true;
    }
    if (p->mode == ZNN_DIRECT)
        return pass == ZNN_PASS_FWD ? direct_fwd(g, a, b, result, ws, s)
             : pass == ZNN_PASS_BWD ? direct_bwd(g, a, b, result, ws, s) : direct_wgrad(g, a, b, result, ws, s);
    if (pass == ZNN_PASS_FWD) return run_fft_fwd(g, way_of(p), a, K, result, ws, memo, s, finish);
    if (pass == ZNN_PASS_WGRAD) return run_fft_wgrad(g, way_of(p), a, b, result, ws, s);
    return run_fft_bwd(g, way_of(p), a, K, result, ws, memo ? memo_gradients(g, way_of(p), memo) : nullptr, s, finish,
                       TileGrad{memo, more ? more->gw : nullptr});
}

bool plan_joins_gradient(const znn_plan* p)
{
    if (p->mode != ZNN_FFT || !p->tile.on) return false;
    const size_t bytes = tile_joined_bytes(p->g, p->tile);
    return bytes && bytes <= plan_pass_bytes(p, ZNN_PASS_WGRAD, false);
}

size_t plan_forward_least(const znn_plan* p)
{
    if (p->mode == ZNN_DIRECT) return direct_fwd_least(p->g);
    return p->tile.on ? fft_workspace(p->g, p->fold, ZNN_PASS_FWD, p->resident != nullptr).total
                      : plan_pass_bytes(p, ZNN_PASS_FWD, p->resident != nullptr);
}

int plan_forward_within(znn_plan* p, const float* in, const float* w, float* out, void* ws, size_t bytes, hipStream_t s)
{
    if (p->mode == ZNN_DIRECT && w && direct_workspace_bytes(p->g, ZNN_PASS_FWD) > bytes) return direct_fwd_groups(p->g, in, w, out, ws, s);
    if (!p->tile.on) return znn_conv3d_fwd(p, in, w, out, ws, bytes, s);
    if (!w && !p->resident) return fail(ZNN_EINVAL, "kernel pointer is NULL");
    const int rc = tile_fwd(p->g, p->tile, in, KernelSpectra{w, p->resident, nullptr}, out, ws, bytes, p->memo, Finish{}, s);
    if (p->memo) p->memo_has_in = rc == ZNN_OK;
    return rc;
}

int plan_wgrad_memo(const znn_plan* p, float2* memo, float* gw, void* ws, hipStream_t s)
{
    return run_fft_wgrad_from_spectra(p->g, way_of(p), memo, memo_gradients(p->g, way_of(p), memo), gw, ws, s);
}

static bool aligned256(const void* p) { return ((uintptr_t)p & 255) == 0; }

static int check_ws(const znn_plan* p, int pass, void* ws, size_t ws_bytes)
{
    size_t need = 0;
    int rc = znn_plan_workspace_bytes(p, pass, &need);
    if (rc != ZNN_OK) return rc;
    if (need == 0) return ZNN_OK;
    if (!ws) return fail(ZNN_EWORKSPACE, "workspace is NULL but %zu bytes are needed", need);
    if (!aligned256(ws)) return fail(ZNN_EWORKSPACE, "workspace is not 256-byte aligned");
    if (ws_bytes < need) return fail(ZNN_EWORKSPACE, "workspace has %zu bytes, %zu needed", ws_bytes, need);
    return ZNN_OK;
}

}  // namespace znn

using namespace znn;

extern "C" {

const char* znn_last_error(void) { return g_err; }

int znn_trace_enable(int32_t on)
{
    std::lock_guard<std::mutex> lk(g_trace_mu);
    g_trace_on = on != 0;
    return ZNN_OK;
}

int znn_trace_collect(znn_trace_record* records, int32_t capacity, int32_t* count)
{
    if (!count || capacity < 0 || (capacity > 0 && !records)) return fail(ZNN_EINVAL, "bad trace buffer");
    std::lock_guard<std::mutex> lk(g_trace_mu);
    int n = 0, rc = ZNN_OK;
    for (TraceEntry& e : g_trace) {
        float ms = 0.f;
        if (hipEventSynchronize(e.e1) != hipSuccess || hipEventElapsedTime(&ms, e.e0, e.e1) != hipSuccess)
            rc = fail(ZNN_EHIP, "cannot read the events of '%s'", e.name);
        if (n < capacity) {
            snprintf(records[n].name, sizeof(records[n].name), "%s", e.name);
            records[n].ms = ms;
        }
        ++n;
        (void)hipEventDestroy(e.e0);
        (void)hipEventDestroy(e.e1);
    }
    g_trace.clear();
    *count = n;
    return rc;
}

int znn_plan_create(const znn_conv_desc* desc, znn_plan** plan)
{
    if (!plan) return fail(ZNN_EINVAL, "plan output pointer is NULL");
    Geom g;
    int rc = validate_desc(desc, &g);
    if (rc != ZNN_OK) return rc;
    int mode = desc->mode;
    if (mode == ZNN_AUTO) {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        auto it = g_tune.find(key_of(*desc));
        mode = (it != g_tune.end()) ? it->second : model_choice(g);
        if (mode == ZNN_FFT && (g.Nz > kMaxFftExtent || g.Ny > kMaxFftExtent || g.Nx > kMaxFftExtent))
            mode = ZNN_DIRECT;
    }
    if (mode == ZNN_FFT && (g.Nz > kMaxFftExtent || g.Ny > kMaxFftExtent || g.Nx > kMaxFftExtent))
        return fail(ZNN_EUNSUPPORTED, "FFT extents above %d are not supported", kMaxFftExtent);
    znn_plan* p = new (std::nothrow) znn_plan;
    if (!p) return fail(ZNN_EINVAL, "out of host memory");
    p->desc = *desc;
    p->g = g;
    p->mode = mode;
    const FftWay way = mode == ZNN_FFT ? fft_way(g) : FftWay{fold_full(), Tiling{}};
    p->fold = way.fold;
    p->tile = way.tile;
    p->resident = nullptr;
    p->memo = nullptr;
    p->memo_bytes = 0;
    p->memo_has_in = p->memo_has_gout = false;
    p->round_memory = SIZE_MAX;
    *plan = p;
    return ZNN_OK;
}

void znn_plan_destroy(znn_plan* plan) { delete plan; }

int znn_plan_mode(const znn_plan* plan, int32_t* mode)
{
    if (!plan || !mode) return fail(ZNN_EINVAL, "NULL argument");
    *mode = plan->mode;
    return ZNN_OK;
}

int znn_plan_fft_extents(const znn_plan* plan, znn_vec3* N)
{
    if (!plan || !N) return fail(ZNN_EINVAL, "NULL argument");
    N->z = plan->g.Nz; N->y = plan->g.Ny; N->x = plan->g.Nx;
    return ZNN_OK;
}

int znn_plan_workspace_bytes(const znn_plan* plan, int32_t pass, size_t* bytes)
{
    if (!plan || !bytes) return fail(ZNN_EINVAL, "NULL argument");
    if (pass < ZNN_PASS_FWD || pass > ZNN_PASS_WGRAD) return fail(ZNN_EINVAL, "unknown pass %d", pass);
    *bytes = plan_pass_bytes(plan, pass, plan->resident != nullptr);
    return ZNN_OK;
}

int znn_plan_set_round_memory(znn_plan* plan, size_t bytes)
{
    if (!plan) return fail(ZNN_EINVAL, "plan is NULL");
    plan->round_memory = bytes;
    return ZNN_OK;
}

int znn_plan_spectra_bytes(const znn_plan* plan, size_t* bytes)
{
    if (!plan || !bytes) return fail(ZNN_EINVAL, "NULL argument");
    *bytes = fft_spectra_bytes(plan->g, plan->fold);
    return ZNN_OK;
}

int znn_plan_tiles(const znn_plan* plan, znn_vec3* length, znn_vec3* count)
{
    if (!plan || !length || !count) return fail(ZNN_EINVAL, "NULL argument");
    const Tiling& L = plan->tile;
    *length = L.on ? znn_vec3{L.M[0], L.M[1], L.M[2]} : znn_vec3{0, 0, 0};
    *count = L.on ? znn_vec3{L.T[0], L.T[1], L.T[2]} : znn_vec3{0, 0, 0};
    return ZNN_OK;
}

int znn_plan_spectra_layout(const znn_plan* plan, int32_t* layout)
{
    if (!plan || !layout) return fail(ZNN_EINVAL, "NULL argument");
    *layout = plan->fold.on ? ZNN_SPECTRA_FOLDED : ZNN_SPECTRA_FULL;
    return ZNN_OK;
}

int znn_plan_set_spectra_layout(znn_plan* plan, int32_t layout)
{
    if (!plan) return fail(ZNN_EINVAL, "NULL argument");
    if (plan->mode != ZNN_FFT) return fail(ZNN_EINVAL, "kernel spectra exist only for the FFT method");
    if (plan->resident)
        return fail(ZNN_EINVAL, "resident kernel spectra are attached in the current layout; release them first");
    if (layout == ZNN_SPECTRA_AUTO) {
        FftWay way = fft_way(plan->g);
        // an attached memo buffer that was sized for whole volumes keeps them
        if (plan->memo && plan->memo_bytes < fft_memo_bytes(plan->g, way)) way.tile.on = false;
        plan->fold = way.fold;
        plan->tile = way.tile;
    } else if (layout == ZNN_SPECTRA_FULL) { plan->fold = fold_full(); plan->tile.on = false; }
    else if (layout == ZNN_SPECTRA_FOLDED) {
        const Fold F = fold_forced(plan->g);
        if (!F.on)
            return fail(ZNN_EUNSUPPORTED, "half spectra need a slowest axis whose FFT extent is divisible by 4 "
                                          "with at most %d taps one voxel apart", kMaxFoldedTaps);
        plan->fold = F;
        plan->tile.on = false;
    } else return fail(ZNN_EINVAL, "unknown spectra layout %d", layout);
    plan->memo_has_in = plan->memo_has_gout = false;    // spectra of another layout
    return ZNN_OK;
}

int znn_conv_prepare_kernels(znn_plan* plan, const float* w, void* spectra, size_t spectra_bytes,
                             void* ws, size_t ws_bytes, void* stream)
{
    (void)ws; (void)ws_bytes;
    if (!plan || !w) return fail(ZNN_EINVAL, "NULL argument");
    if (plan->mode != ZNN_FFT) return fail(ZNN_EINVAL, "kernel spectra exist only for the FFT method");
    const size_t need = fft_spectra_bytes(plan->g, plan->fold);
    if (!spectra) return fail(ZNN_EWORKSPACE, "spectra buffer is NULL");
    if (!aligned256(spectra)) return fail(ZNN_EWORKSPACE, "spectra buffer is not 256-byte aligned");
    if (spectra_bytes < need) return fail(ZNN_EWORKSPACE, "spectra buffer has %zu bytes, %zu needed", spectra_bytes, need);
    int rc = run_kernel_spectra(plan->g, way_of(plan), w, (float2*)spectra, (hipStream_t)stream);
    if (rc != ZNN_OK) return rc;
    plan->resident = (const float2*)spectra;
    return ZNN_OK;
}

int znn_plan_memo_bytes(const znn_plan* plan, size_t* bytes)
{
    if (!plan || !bytes) return fail(ZNN_EINVAL, "NULL argument");
    *bytes = fft_memo_bytes(plan->g, way_of(plan));
    return ZNN_OK;
}

int znn_conv_set_memo(znn_plan* plan, void* memo, size_t memo_bytes)
{
    if (!plan) return fail(ZNN_EINVAL, "NULL argument");
    plan->memo = nullptr;
    plan->memo_has_in = plan->memo_has_gout = false;
    if (!memo) return ZNN_OK;
    if (plan->mode != ZNN_FFT) return fail(ZNN_EINVAL, "spectra are memoized only by the FFT method");
    size_t need = 0;
    znn_plan_memo_bytes(plan, &need);
    if (!aligned256(memo)) return fail(ZNN_EWORKSPACE, "memo buffer is not 256-byte aligned");
    if (memo_bytes < need) return fail(ZNN_EWORKSPACE, "memo buffer has %zu bytes, %zu needed", memo_bytes, need);
    plan->memo = (float2*)memo;
    plan->memo_bytes = memo_bytes;
    return ZNN_OK;
}

int znn_conv3d_wgrad_memo(znn_plan* plan, float* gw, void* ws, size_t ws_bytes, void* stream)
{
    if (!plan || !gw) return fail(ZNN_EINVAL, "NULL argument");
    if (plan->mode != ZNN_FFT || !plan->memo) return fail(ZNN_EINVAL, "no memo buffer is attached to this plan");
    if (!plan->memo_has_in || !plan->memo_has_gout)
        return fail(ZNN_EINVAL, "the forward and the backward pass must run on this plan first");
    int rc = check_ws(plan, ZNN_PASS_WGRAD, ws, ws_bytes);
    if (rc != ZNN_OK) return rc;
    return plan_wgrad_memo(plan, plan->memo, gw, ws, (hipStream_t)stream);
}

int znn_conv_release_kernels(znn_plan* plan)
{
    if (!plan) return fail(ZNN_EINVAL, "NULL argument");
    plan->resident = nullptr;
    return ZNN_OK;
}

int znn_conv3d_fwd(znn_plan* plan, const float* in, const float* w, float* out,
                   void* ws, size_t ws_bytes, void* stream)
{
    if (!plan || !in || !out) return fail(ZNN_EINVAL, "NULL argument");
    if (!w && !(plan->mode == ZNN_FFT && plan->resident)) return fail(ZNN_EINVAL, "kernel pointer is NULL");
    int rc = check_ws(plan, ZNN_PASS_FWD, ws, ws_bytes);
    if (rc != ZNN_OK) return rc;
    rc = plan_pass(plan, ZNN_PASS_FWD, in, w, out, plan->resident, ws, plan->memo, (hipStream_t)stream);
    if (plan->memo) plan->memo_has_in = rc == ZNN_OK;
    return rc;
}

int znn_conv3d_bwd(znn_plan* plan, const float* gout, const float* w, float* gin,
                   void* ws, size_t ws_bytes, void* stream)
{
    if (!plan || !gout || !gin) return fail(ZNN_EINVAL, "NULL argument");
    if (!w && !(plan->mode == ZNN_FFT && plan->resident)) return fail(ZNN_EINVAL, "kernel pointer is NULL");
    int rc = check_ws(plan, ZNN_PASS_BWD, ws, ws_bytes);
    if (rc != ZNN_OK) return rc;
    rc = plan_pass(plan, ZNN_PASS_BWD, gout, w, gin, plan->resident, ws, plan->memo, (hipStream_t)stream);
    if (plan->memo) plan->memo_has_gout = rc == ZNN_OK;
    return rc;
}

int znn_conv3d_wgrad(znn_plan* plan, const float* in, const float* gout, float* gw,
                     void* ws, size_t ws_bytes, void* stream)
{
    if (!plan || !in || !gout || !gw) return fail(ZNN_EINVAL, "NULL argument");
    int rc = check_ws(plan, ZNN_PASS_WGRAD, ws, ws_bytes);
    if (rc != ZNN_OK) return rc;
    return plan_pass(plan, ZNN_PASS_WGRAD, in, gout, gw, nullptr, ws, nullptr, (hipStream_t)stream);
}

// ---------------------------------------------------------------- autotuner
static size_t tune_tensor_bytes(const Geom& g, size_t off[6])
{
    size_t o = 0;
    off[0] = o; o += align256(sizeof(float) * g.f * g.nvol());                 // in
    off[1] = o; o += align256(sizeof(float) * g.fo * g.f * g.kvol());          // w
    off[2] = o; o += align256(sizeof(float) * g.fo * g.ovol());                // gout
    off[3] = o; o += align256(sizeof(float) * g.f * g.nvol());                 // gin
    off[4] = o; o += align256(sizeof(float) * g.fo * g.f * g.kvol());          // gw
    off[5] = o; o += align256(sizeof(float) * g.fo * g.ovol());                // out
    return o;
}

static size_t tune_scratch_bytes(const Geom& g, bool fft_ok)
{
    const FftWay F = fft_way(g);
    size_t m = 0;
    for (int pass = 0; pass < 3; ++pass) {
        size_t d = direct_workspace_bytes(g, pass);
        if (d > m) m = d;
        if (fft_ok) {
            size_t f = fft_pass_bytes(g, F, pass, false);
            if (f > m) m = f;
        }
    }
    return m;
}

int znn_autotune_workspace_bytes(const znn_conv_desc* desc, size_t* bytes)
{
    if (!bytes) return fail(ZNN_EINVAL, "NULL argument");
    Geom g;
    int rc = validate_desc(desc, &g);
    if (rc != ZNN_OK) return rc;
    const bool fft_ok = g.Nz <= kMaxFftExtent && g.Ny <= kMaxFftExtent && g.Nx <= kMaxFftExtent;
    size_t off[6];
    *bytes = tune_tensor_bytes(g, off) + tune_scratch_bytes(g, fft_ok);
    return ZNN_OK;
}

int znn_autotune(const znn_conv_desc* desc, void* ws, size_t ws_bytes, void* stream,
                 int32_t* chosen_mode, float ms[2][3])
{
    if (!chosen_mode || !ms) return fail(ZNN_EINVAL, "NULL argument");
    Geom g;
    int rc = validate_desc(desc, &g);
    if (rc != ZNN_OK) return rc;
    const bool fft_ok = g.Nz <= kMaxFftExtent && g.Ny <= kMaxFftExtent && g.Nx <= kMaxFftExtent;
    size_t off[6];
    const size_t tensors = tune_tensor_bytes(g, off);
    const size_t scratch = tune_scratch_bytes(g, fft_ok);
    if (!ws) return fail(ZNN_EWORKSPACE, "workspace is NULL");
    if (!aligned256(ws)) return fail(ZNN_EWORKSPACE, "workspace is not 256-byte aligned");
    if (ws_bytes < tensors + scratch)
        return fail(ZNN_EWORKSPACE, "workspace has %zu bytes, %zu needed", ws_bytes, tensors + scratch);
    hipStream_t s = (hipStream_t)stream;
    char* base = (char*)ws;
    float* in = (float*)(base + off[0]);
    float* w = (float*)(base + off[1]);
    float* gout = (float*)(base + off[2]);
    float* gin = (float*)(base + off[3]);
    float* gw = (float*)(base + off[4]);
    float* out = (float*)(base + off[5]);
    void* scr = base + tensors;
    if ((rc = fill_pattern(in, (long)g.f * g.nvol(), 1.0f, s)) != ZNN_OK) return rc;
    if ((rc = fill_pattern(w, (long)g.fo * g.f * g.kvol(), 1.0f / std::sqrt((float)(g.f * g.kvol())), s)) != ZNN_OK) return rc;
    if ((rc = fill_pattern(gout, (long)g.fo * g.ovol(), 1.0f, s)) != ZNN_OK) return rc;

    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
        return fail(ZNN_EHIP, "hipEventCreate failed");
    const int warm = 2, timed = 5;
    const FftWay F = fft_way(g);
    for (int m = 0; m < 2; ++m)
        for (int p = 0; p < 3; ++p) ms[m][p] = INFINITY;
    rc = ZNN_OK;
    for (int mode = 0; mode < 2 && rc == ZNN_OK; ++mode) {
        if (mode == ZNN_FFT && !fft_ok) continue;
        for (int pass = 0; pass < 3 && rc == ZNN_OK; ++pass) {
            for (int it = 0; it < warm + timed && rc == ZNN_OK; ++it) {
                if (it == warm) (void)hipEventRecord(e0, s);
                if (mode == ZNN_DIRECT) {
                    if (pass == 0) rc = direct_fwd(g, in, w, out, scr, s);
                    else if (pass == 1) rc = direct_bwd(g, gout, w, gin, scr, s);
                    else rc = direct_wgrad(g, in, gout, gw, scr, s);
                } else {
                    if (pass == 0) rc = run_fft_fwd(g, F, in, KernelSpectra{w, nullptr, nullptr}, out, scr, nullptr, s);
                    else if (pass == 1) rc = run_fft_bwd(g, F, gout, KernelSpectra{w, nullptr, nullptr}, gin, scr, nullptr, s);
                    else rc = run_fft_wgrad(g, F, in, gout, gw, scr, s);
                }
            }
            if (rc != ZNN_OK) break;
            (void)hipEventRecord(e1, s);
            if (hipEventSynchronize(e1) != hipSuccess) { rc = fail(ZNN_EHIP, "hipEventSynchronize failed"); break; }
            float t = 0.f;
            (void)hipEventElapsedTime(&t, e0, e1);
            ms[mode][pass] = t / timed;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != ZNN_OK) return rc;
    const float td = ms[0][0] + ms[0][1] + ms[0][2];
    const float tf = ms[1][0] + ms[1][1] + ms[1][2];
    const int choice = (fft_ok && tf < td) ? ZNN_FFT : ZNN_DIRECT;
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        g_tune[key_of(*desc)] = choice;
    }
    *chosen_mode = choice;
    return ZNN_OK;
}

// ---- whole-round strategies under a memory budget (Section 4, memoization)
struct RoundNeeds {
    size_t scratch[3];      // workspace, kernel spectra, memoized node spectra per strategy (summed below)
    size_t total[3];
};

static RoundNeeds round_needs(const Geom& g, bool fft_ok)
{
    RoundNeeds r = {};
    const FftWay F = fft_way(g);
    size_t d = 0, f = 0, fm = 0;
    for (int pass = 0; pass < 3; ++pass) {
        d = std::max(d, direct_workspace_bytes(g, pass));
        if (fft_ok) {
            f = std::max(f, fft_pass_bytes(g, F, pass, false));
            fm = std::max(fm, fft_pass_bytes(g, F, pass, true));
        }
    }
    r.total[ZNN_STRATEGY_DIRECT] = d;
    r.total[ZNN_STRATEGY_FFT] = f;
    r.total[ZNN_STRATEGY_FFT_MEMO] = fft_ok
        ? fm + fft_spectra_bytes(g, F.fold) + fft_memo_bytes(g, F) : 0;
    return r;
}

int znn_autotune_round_workspace_bytes(const znn_conv_desc* desc, size_t* bytes)
{
    if (!bytes) return fail(ZNN_EINVAL, "NULL argument");
    Geom g;
    int rc = validate_desc(desc, &g);
    if (rc != ZNN_OK) return rc;
    const bool fft_ok = g.Nz <= kMaxFftExtent && g.Ny <= kMaxFftExtent && g.Nx <= kMaxFftExtent;
    const RoundNeeds need = round_needs(g, fft_ok);
    size_t off[6];
    *bytes = tune_tensor_bytes(g, off) + std::max(need.total[0], std::max(need.total[1], need.total[2]));
    return ZNN_OK;
}

int znn_autotune_round(const znn_conv_desc* desc, uint64_t memory_budget, void* ws, size_t ws_bytes,
                       void* stream, znn_round_report* report)
{
    if (!report) return fail(ZNN_EINVAL, "NULL argument");
    Geom g;
    int rc = validate_desc(desc, &g);
    if (rc != ZNN_OK) return rc;
    const bool fft_ok = g.Nz <= kMaxFftExtent && g.Ny <= kMaxFftExtent && g.Nx <= kMaxFftExtent;
    const RoundNeeds need = round_needs(g, fft_ok);
    bool run[3];
    size_t scratch = 0;
    int candidates = 0;
    for (int t = 0; t < 3; ++t) {
        report->ms[t] = INFINITY;
        report->bytes[t] = need.total[t];
        run[t] = (t == ZNN_STRATEGY_DIRECT || fft_ok) && need.total[t] <= memory_budget;
        if (run[t]) { scratch = std::max(scratch, need.total[t]); ++candidates; }
    }
    report->chosen = -1;
    if (!candidates)
        return fail(ZNN_EWORKSPACE, "no strategy fits the memory budget of %llu bytes (direct needs %zu)",
                    (unsigned long long)memory_budget, need.total[0]);
    size_t off[6];
    const size_t tensors = tune_tensor_bytes(g, off);
    if (!ws) return fail(ZNN_EWORKSPACE, "workspace is NULL");
    if (!aligned256(ws)) return fail(ZNN_EWORKSPACE, "workspace is not 256-byte aligned");
    if (ws_bytes < tensors + scratch)
        return fail(ZNN_EWORKSPACE, "workspace has %zu bytes, %zu needed", ws_bytes, tensors + scratch);
    hipStream_t s = (hipStream_t)stream;
    char* base = (char*)ws;
    float* in = (float*)(base + off[0]);
    float* w = (float*)(base + off[1]);
    float* gout = (float*)(base + off[2]);
    float* gin = (float*)(base + off[3]);
    float* gw = (float*)(base + off[4]);
    float* out = (float*)(base + off[5]);
    char* scr = base + tensors;
    if ((rc = fill_pattern(in, (long)g.f * g.nvol(), 1.0f, s)) != ZNN_OK) return rc;
    if ((rc = fill_pattern(w, (long)g.fo * g.f * g.kvol(), 1.0f / std::sqrt((float)(g.f * g.kvol())), s)) != ZNN_OK) return rc;
    if ((rc = fill_pattern(gout, (long)g.fo * g.ovol(), 1.0f, s)) != ZNN_OK) return rc;
    // memoized strategy: [pass workspace | kernel spectra | node spectra]
    const FftWay F = fft_way(g);
    size_t memo_ws = 0;
    if (fft_ok)
        for (int pass = 0; pass < 3; ++pass) memo_ws = std::max(memo_ws, fft_pass_bytes(g, F, pass, true));
    float2* What = (float2*)(scr + memo_ws);
    float2* Ihat = (float2*)(scr + memo_ws + fft_spectra_bytes(g, F.fold));
    float2* Ghat = memo_gradients(g, F, Ihat);

    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
        return fail(ZNN_EHIP, "hipEventCreate failed");
    const int warm = 2, timed = 5;
    for (int t = 0; t < 3 && rc == ZNN_OK; ++t) {
        if (!run[t]) continue;
        for (int it = 0; it < warm + timed && rc == ZNN_OK; ++it) {
            if (it == warm) (void)hipEventRecord(e0, s);
            if (t == ZNN_STRATEGY_DIRECT) {
                rc = direct_fwd(g, in, w, out, scr, s);
                if (rc == ZNN_OK) rc = direct_bwd(g, gout, w, gin, scr, s);
                if (rc == ZNN_OK) rc = direct_wgrad(g, in, gout, gw, scr, s);
            } else if (t == ZNN_STRATEGY_FFT) {
                rc = run_fft_fwd(g, F, in, KernelSpectra{w, nullptr, nullptr}, out, scr, nullptr, s);
                if (rc == ZNN_OK) rc = run_fft_bwd(g, F, gout, KernelSpectra{w, nullptr, nullptr}, gin, scr, nullptr, s);
                if (rc == ZNN_OK) rc = run_fft_wgrad(g, F, in, gout, gw, scr, s);
            } else {
                rc = run_kernel_spectra(g, F, w, What, s);
                if (rc == ZNN_OK) rc = run_fft_fwd(g, F, in, KernelSpectra{nullptr, What, nullptr}, out, scr, Ihat, s);
                if (rc == ZNN_OK) rc = run_fft_bwd(g, F, gout, KernelSpectra{nullptr, What, nullptr}, gin, scr, Ghat, s);
                if (rc == ZNN_OK) rc = run_fft_wgrad_from_spectra(g, F, Ihat, Ghat, gw, scr, s);
            }
        }
        if (rc != ZNN_OK) break;
        (void)hipEventRecord(e1, s);
        if (hipEventSynchronize(e1) != hipSuccess) { rc = fail(ZNN_EHIP, "hipEventSynchronize failed"); break; }
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, e0, e1);
        report->ms[t] = ms / timed;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != ZNN_OK) return rc;
    int best = -1;
    for (int t = 0; t < 3; ++t)
        if (run[t] && (best < 0 || report->ms[t] < report->ms[best])) best = t;
    report->chosen = best;
    {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        g_tune[key_of(*desc)] = best == ZNN_STRATEGY_DIRECT ? ZNN_DIRECT : ZNN_FFT;
    }
    return ZNN_OK;
}

}  // extern "C"
