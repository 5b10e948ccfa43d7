// A round of a net as one native call: the passes of all layers are put in order once (znn_program_create) and then
// launched back to back from here (znn_program_run).
//
// Rounds of small and ordinary nets were bound by their launches: 78 of them for the six-layer 3D net, issued at 8 us each
// where every one is a call from the host language.  A program
//   * issues its launches natively (about 2 us each) on the given streams, with the events between streams derived
//     from the buffers that its steps read and write;
//   * packs the weights of all direct convolutions in one launch (k_pack_weights);
//   * lets the kernel that completes an image also apply the transfer function of the next edge, and the kernel that
//     completes a backward image the derivative of the edge below (conv::Finish, k_finish_fwd, k_finish_bwd, max-filter);
//   * sums the biases' gradients of all layers in one launch that fills the chip (k_bias_parts: one workgroup per
//     map and 8192 voxels; one workgroup per map took 76 us on the sparse net), and in the last launch completes
//     the sums of all kernel and bias gradients and updates all parameters (k_update);
//   * keeps the spectra of a layer on the FFT method from the forward to the backward pass and the gradient;
//   * on one stream, copies the images of the kernel gradients of small layers by one launch at the end, takes the gradients on the vector
//     ALUs and the biases' sums by another, and those of small FFT layers by the launches of their backward passes.
// Six-layer 3D net on a 12^3 patch: 78 -> 31 launches, 617 -> 413 us on the fp32 direct kernels, 268 us on those on split operands: chains
// of kernels of 4 to 26 us (direct passes 144 us, gradients with their copies and sums 85 us, the rest 2 to 9 us each).
#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include "bias_parts.h"
#include "znn_internal.h"

namespace znn {

namespace {

__device__ __forceinline__ float derivative_times(int fn, float g, float y)
{
    if (fn == ZNN_RECTIFY) return y > 0.f ? g : 0.f;
    return g * (fn == ZNN_LOGISTIC ? y * (1.0f - y) : 1.0f - y * y);
}

__device__ __forceinline__ float transfer(int fn, float v)
{
    if (fn == ZNN_RECTIFY) return v > 0.f ? v : 0.f;
    return fn == ZNN_LOGISTIC ? 1.0f / (1.0f + expf(-v)) : tanhf(v);
}

// x = sum of the shares in ascending order (k_conv_reduce), y = fn(x + bias).  blockIdx.y: map.
__global__ void __launch_bounds__(256)
k_finish_fwd(const float* __restrict__ partial, float* __restrict__ x, const float* __restrict__ bias, float* __restrict__ y,
             int voxels, long count, int splits, int fn)
{
    const int v = blockIdx.x * 256 + threadIdx.x;
    if (v >= voxels) return;
    const long t = (long)blockIdx.y * voxels + v;
    float acc = partial[t];
#pragma unroll 4
    for (int s = 1; s < splits; ++s) acc += partial[(long)s * count + t];
    x[t] = acc;
    y[t] = transfer(fn, acc + bias[blockIdx.y]);
}

// g = (sum of the shares) times the derivative of the transfer function that gave y
__global__ void __launch_bounds__(256)
k_finish_bwd(const float* __restrict__ partial, const float* __restrict__ y, float* __restrict__ g, long count, int splits, int fn)
{
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    if (t >= count) return;
    float acc = partial[t];
#pragma unroll 4
    for (int s = 1; s < splits; ++s) acc += partial[(long)s * count + t];
    g[t] = derivative_times(fn, acc, y[t]);
}

__global__ void __launch_bounds__(256) k_derivative_in_place(float* g, const float* __restrict__ y, long count, int fn)
{
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    if (t < count) g[t] = derivative_times(fn, g[t], y[t]);
}

// Loss gradient and, for the output edge below it, the gradient before the transfer function (gx may be NULL).
__global__ void __launch_bounds__(256)
k_loss_finish(long count, const float* __restrict__ y, const float* __restrict__ target, float* __restrict__ g,
              float* __restrict__ gx, int loss, int fn)
{
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    if (t >= count) return;
    const float v = y[t];
    const float e = loss == ZNN_LOSS_SQUARE ? v - target[t] : (v - target[t]) / (v * (1.0f - v));
    g[t] = e;
    if (gx) gx[t] = derivative_times(fn, e, v);
}

// Node sums: the parts in ascending order, times the derivative of the edge below if y is given.
struct SumArgs { const float* part[6]; const float* y; float* out; long count; int parts, fn; };
__global__ void __launch_bounds__(256) k_node_sum(SumArgs A)
{
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    if (t >= A.count) return;
    float acc = A.part[0][t];
    for (int i = 1; i < A.parts; ++i) acc = acc + A.part[i][t];
    A.out[t] = A.y ? derivative_times(A.fn, acc, A.y[t]) : acc;
}

// Sums of the gradients over the voxels of every map.
constexpr int kBiasItems = 64;
struct BiasArgs { BiasItem item[kBiasItems]; int n; };
__global__ void __launch_bounds__(256) k_bias_parts(BiasArgs A)
{
    __shared__ float red[4];
    int q = 0;
    while (q + 1 < A.n && blockIdx.x >= A.item[q + 1].first) ++q;       // uniform
    bias_part(A.item[q], blockIdx.x - A.item[q].first, red);
}

// Completes the gradients of a round and updates the parameters.  An item is the kernels or the biases of a layer:
//   kind 0: the gradient is there;  kind 1: shares of the direct kernel gradient, in the order of k_wgrad_sum;
//   kind 2: the same in the order of k_wgrad_sum4 (four waves per 64 elements);  kind 3: `spans` parts per bias.
// p may be NULL (gradient only).
constexpr int kUpdateItems = 32;
struct UpdateItem {
    const float* src; float* grad; float* p;
    long total; unsigned first;
    int kind;
    WgradSum sum;           // kind 3: sum.ksplit parts
};
struct UpdateArgs { UpdateItem item[kUpdateItems]; int n; float eta; };
__global__ void __launch_bounds__(256) k_update(UpdateArgs A)
{
    __shared__ float part[4][64];
    int q = 0;
    while (q + 1 < A.n && blockIdx.x >= A.item[q + 1].first) ++q;       // uniform
    const UpdateItem& U = A.item[q];
    const unsigned r = blockIdx.x - U.first;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const bool shares = U.kind == 1 || U.kind == 2;         // threads run along the partial sums
    const long e = U.kind == 2 ? (long)r * 64 + lane : (long)r * 256 + threadIdx.x;
    long t = e, from = 0;
    const bool live = shares ? e < U.sum.slots && wgrad_slot(U.sum, e, from, t) : e < U.total;
    float acc = 0.f;
    if (live) {
        const int n = U.sum.ksplit;
        if (U.kind == 0) acc = U.grad[t];
        else if (U.kind == 3) for (int s = 0; s < n; ++s) acc += U.src[t * n + s];
        else {
            const float* p = U.src + from;
            const long step = (long)U.sum.planes * U.sum.Mpad * U.sum.Npad;
            if (U.kind == 1) {
#pragma unroll 4
                for (int s = 0; s < n; ++s) acc += p[s * step];
            } else {
#pragma unroll 4
                for (int s = wave; s < n; s += 4) acc += p[s * step];
            }
        }
    }
    if (U.kind == 2) {      // uniform
        part[wave][lane] = acc;
        __syncthreads();
        if (wave != 0) return;
        acc = ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
    }
    if (!live) return;
    if (U.kind != 0) U.grad[t] = acc;
    if (U.p) U.p[t] = U.p[t] - A.eta * acc;
}

// A step of the program: an operation of the caller, or one of five that the program adds.
enum { STEP_PACK = -1, STEP_BIAS = -2, STEP_UPDATE = -3, STEP_GRADS = -4, STEP_FEW = -5 };
constexpr size_t kNone = (size_t)-1;

struct Step {
    int kind;
    znn_op op;
    int stream;
    bool skip;                          // no launch of its own: part of STEP_GRADS, STEP_FEW, STEP_BIAS or STEP_UPDATE, or of the backward pass
    int layer;                          // convolutions: index into znn_program::layers
    size_t own;                         // place of the partial sums that STEP_UPDATE completes (kNone: it writes the gradient)
    size_t copies;                      // kernel gradients of STEP_GRADS: place of their copies
    size_t pass_bytes;                  // scratch it needs while it runs
    WgradSum sum;
    std::vector<int> reads, writes;     // resources
    std::vector<int> waits;             // steps of other streams that must be over
    hipEvent_t event;                   // recorded behind the step if another stream waits for it
};

// What the program keeps of a plan (the plan as it was when the program was made).
struct Layer {
    const znn_plan* of;
    znn_plan plan;
    int w, in, gout;        // its buffers
    int step[3];            // its passes: steps of this program, -1 where there is none
    size_t packed[2];       // direct method: weights of the forward / backward pass from the round's packing launch
    size_t spectra;         // FFT method: kernels, transformed once, by the first of the two passes that use them
    size_t memo;            // and the spectra of images and gradients, kept for a kernel gradient that comes after both
    bool joined;            // the kernel gradient is made by the launches of the backward pass
};

long elements(const znn_op& o) { return (long)o.maps * o.n.z * o.n.y * o.n.x; }
long voxels(const znn_op& o) { return (long)o.n.z * o.n.y * o.n.x; }
int bias_spans(const znn_op& o) { return (int)((voxels(o) + kBiasSpan - 1) / kBiasSpan); }

}  // namespace

}  // namespace znn

using namespace znn;

struct znn_program {
    int buffers, streams;
    std::vector<Layer> layers;
    std::vector<Step> steps;
    std::vector<int> last_waits;        // steps that stream 0 waits for at the end
    std::vector<char> used;             // streams with work on them
    hipEvent_t start;
    size_t scratch;
    std::vector<size_t> area;           // per stream: place of the scratch of its passes
    std::vector<int> bias_steps;        // deferred bias gradients
    std::vector<int> grad_steps;        // kernel gradients whose images are copied by one launch
    std::vector<int> few_steps;         // kernel gradients on the vector ALUs that share a launch, with the bias gradients
    std::vector<int> update_steps;
    std::vector<int> completes;         // per update: the step whose sums it completes, or -1
};

namespace znn {

namespace {

// spectra that a program keeps on the device between the passes of a round, at most
constexpr size_t kKeptSpectra = (size_t)16 << 30;

// Per kind, as masks over the positions of znn_op::buf: which must be given, and what the operation reads and writes.
struct Form { unsigned need; int n; unsigned reads, writes; };
constexpr Form kForm[] = {
    {7u, 5, 0x0bu, 0x14u},      // CONV_FWD
    {7u, 4, 0x0bu, 0x04u},      // CONV_BWD
    {7u, 3, 0x03u, 0x04u},      // CONV_WGRAD
    {7u, 3, 0x03u, 0x04u},      // TRANSFER_FWD
    {7u, 3, 0x03u, 0x04u},      // TRANSFER_BWD
    {3u, 2, 0x01u, 0x02u},      // BIAS_GRAD
    {7u, 3, 0x01u, 0x06u},      // FILTER_FWD
    {7u, 4, 0x0bu, 0x04u},      // FILTER_BWD
    {7u, 3, 0x01u, 0x06u},      // POOL_FWD
    {7u, 4, 0x0bu, 0x04u},      // POOL_BWD
    {7u, 4, 0x03u, 0x0cu},      // LOSS_GRAD
    {3u, 8, 0xfeu, 0x01u},      // NODE_SUM
    {3u, 2, 0x03u, 0x02u},      // UPDATE
};

bool uses(const Step& s, unsigned positions, int buffer)
{
    for (int q = 0; q < 8; ++q)
        if ((positions >> q & 1) && s.op.buf[q] == buffer) return true;
    return false;
}

unsigned writes(const Step& s) { return s.kind < 0 ? 0u : kForm[s.kind].writes; }
unsigned touches(const Step& s) { return s.kind < 0 ? 0u : kForm[s.kind].reads | kForm[s.kind].writes; }

// whether a step after `first` and before `last` writes / reads or writes the buffer
bool written_between(const znn_program& P, int buffer, int first, int last)
{
    for (int i = first + 1; i < last; ++i)
        if (uses(P.steps[i], writes(P.steps[i]), buffer)) return true;
    return false;
}

bool touched_between(const znn_program& P, int buffer, int first, int last)
{
    for (int i = first + 1; i < last; ++i)
        if (uses(P.steps[i], touches(P.steps[i]), buffer)) return true;
    return false;
}

int check_op(const znn_op& o, int i, int buffers, int streams)
{
    if (o.kind < ZNN_OP_CONV_FWD || o.kind > ZNN_OP_UPDATE) return fail(ZNN_EINVAL, "operation %d: unknown kind %d", i, o.kind);
    if (o.stream < 0 || o.stream >= streams) return fail(ZNN_EINVAL, "operation %d: no stream %d", i, o.stream);
    const Form& form = kForm[o.kind];
    for (int b = 0; b < 8; ++b) {
        if (o.buf[b] >= buffers) return fail(ZNN_EINVAL, "operation %d: no buffer %d", i, o.buf[b]);
        if (o.buf[b] < 0 && (form.need >> b & 1)) return fail(ZNN_EINVAL, "operation %d: buffer %d is missing", i, b);
        if (o.buf[b] >= 0 && b >= form.n) return fail(ZNN_EINVAL, "operation %d: buffer %d has no meaning", i, b);
    }
    if (o.kind == ZNN_OP_NODE_SUM)
        for (int b = 2; b < 7; ++b)
            if (o.buf[b] >= 0 && o.buf[b - 1] < 0) return fail(ZNN_EINVAL, "operation %d: part %d of the sum is missing", i, b - 1);
    if (o.fn < ZNN_RECTIFY || o.fn > ZNN_TANH) return fail(ZNN_EINVAL, "operation %d: unknown transfer function %d", i, o.fn);
    if (o.kind <= ZNN_OP_CONV_WGRAD) {
        if (!o.plan) return fail(ZNN_EINVAL, "operation %d: plan is NULL", i);
        if (o.kind == ZNN_OP_CONV_FWD && (o.buf[3] < 0) != (o.buf[4] < 0))
            return fail(ZNN_EINVAL, "operation %d: a transfer function needs biases and a result", i);
        return ZNN_OK;
    }
    if (o.kind == ZNN_OP_LOSS_GRAD && o.loss != ZNN_LOSS_SQUARE && o.loss != ZNN_LOSS_CROSS_ENTROPY)
        return fail(ZNN_EINVAL, "operation %d: unknown loss %d", i, o.loss);
    if (o.maps < 1 || o.n.z < 1 || o.n.y < 1 || o.n.x < 1) return fail(ZNN_EINVAL, "operation %d: maps and extents must be >= 1", i);
    if ((double)o.maps * o.n.z * o.n.y * o.n.x / 256 >= 2147483647.0)
        return fail(ZNN_EUNSUPPORTED, "operation %d: too many elements for one launch", i);
    if (o.kind == ZNN_OP_FILTER_FWD || o.kind == ZNN_OP_FILTER_BWD || o.kind == ZNN_OP_POOL_FWD || o.kind == ZNN_OP_POOL_BWD)
        return check_filter(o.maps, o.n, o.window, o.sparsity, o.kind == ZNN_OP_POOL_FWD || o.kind == ZNN_OP_POOL_BWD);
    return ZNN_OK;
}

int layer_of(znn_program& P, const znn_op& o, int i, int step)
{
    size_t l = 0;
    while (l < P.layers.size() && P.layers[l].of != o.plan) ++l;
    if (l == P.layers.size()) {
        Layer L = {};
        L.of = o.plan;
        L.plan = *o.plan;
        L.plan.resident = nullptr; L.plan.memo = nullptr;
        L.w = L.in = L.gout = -1;
        L.step[0] = L.step[1] = L.step[2] = -1;
        L.packed[0] = L.packed[1] = L.spectra = L.memo = kNone;
        P.layers.push_back(L);
    }
    Layer& L = P.layers[l];
    bool same = L.step[o.kind] < 0;
    auto is = [&](int& have, int b) { same = same && (have < 0 || have == b); have = b; };
    if (o.kind != ZNN_OP_CONV_WGRAD) is(L.w, o.buf[1]);
    if (o.kind != ZNN_OP_CONV_BWD) is(L.in, o.buf[0]);
    if (o.kind != ZNN_OP_CONV_FWD) is(L.gout, o.buf[o.kind == ZNN_OP_CONV_BWD ? 0 : 1]);
    L.step[o.kind] = step;
    if (!same) { fail(ZNN_EINVAL, "operation %d: a plan stands for one layer of the program", i); return -1; }
    return (int)l;
}

// Steps, places in the scratch memory and what is completed by the update.
int place_steps(znn_program& P, const znn_op* ops, int count)
{
    auto add = [&](int kind) -> Step& {
        Step s = {};
        s.kind = kind; s.layer = -1; s.own = s.copies = kNone;
        P.steps.push_back(s);
        return P.steps.back();
    };
    add(STEP_PACK).skip = true;
    for (int i = 0; i < count; ++i) {
        int rc = check_op(ops[i], i, P.buffers, P.streams);
        if (rc != ZNN_OK) return rc;
        Step& s = add(ops[i].kind);
        s.op = ops[i];
        s.stream = ops[i].stream;
        if (s.kind <= ZNN_OP_CONV_WGRAD && (s.layer = layer_of(P, ops[i], i, (int)P.steps.size() - 1)) < 0) return ZNN_EINVAL;
    }
    const int n = (int)P.steps.size();
    for (int u = 0; u < n; ++u) {
        if (P.steps[u].kind != ZNN_OP_UPDATE) continue;
        const znn_op& o = P.steps[u].op;
        int i = u - 1;
        while (i >= 0 && !uses(P.steps[i], writes(P.steps[i]), o.buf[0])) --i;
        const Step* made = i < 0 ? nullptr : &P.steps[i];
        const long have = !made ? -1 : made->kind == ZNN_OP_BIAS_GRAD ? made->op.maps
                        : made->kind == ZNN_OP_CONV_WGRAD ? (long)made->op.plan->g.f * made->op.plan->g.fo * made->op.plan->g.kvol() : -1;
        if (have >= 0 && have != elements(o))
            return fail(ZNN_EINVAL, "operation %d: an update of %ld elements from a gradient of %ld", u - 1, elements(o), have);
    }
    std::vector<int> last_touch(P.buffers, -1), last_write(P.buffers, -1);
    for (int i = 0; i < n; ++i)
        for (int q = 0; q < 8; ++q) {
            const Step& s = P.steps[i];
            const int b = s.op.buf[q];
            if (touches(s) >> q & 1 && b >= 0) last_touch[b] = i;
            if (writes(s) >> q & 1 && b >= 0) last_write[b] = i;
        }
    // An update joins the one launch at the end where no operation behind it could tell
    for (int i = 0; i < n; ++i) {
        Step& s = P.steps[i];
        if (s.kind != ZNN_OP_UPDATE || last_touch[s.op.buf[0]] > i || last_touch[s.op.buf[1]] > i) continue;
        s.skip = true;
        P.update_steps.push_back(i);
    }
    size_t at = 0, spectra = 0;
    auto take = [&](size_t bytes) { const size_t o = at; at += align256(bytes); return o; };
    // what a layer may hold besides: its plan's bound, and one on all spectra
    std::vector<size_t> room;
    auto hold = [&](size_t layer, size_t bytes) { return bytes > room[layer] ? kNone : (room[layer] -= bytes, take(bytes)); };
    auto hold_spectra = [&](size_t layer, size_t bytes) {
        if (bytes > kKeptSpectra - spectra || bytes > room[layer]) return kNone;
        spectra += bytes;
        return hold(layer, bytes);
    };
    for (size_t l = 0; l < P.layers.size(); ++l) {
        Layer& L = P.layers[l];
        room.push_back(L.plan.round_memory);
        if (L.plan.mode == ZNN_DIRECT) {
            for (int b = 0; b < 2; ++b)
                if (L.step[b] >= 0 && conv_takes_packed(L.plan.g, b == 1) && !written_between(P, L.w, 0, L.step[b])) {
                    L.packed[b] = hold(l, conv_packed_bytes(L.plan.g, b == 1));
                    if (L.packed[b] != kNone) P.steps[0].skip = false;
                }
        } else if (L.step[0] >= 0 && L.step[1] >= 0) {
            const int fwd = L.step[0], bwd = L.step[1], grad = L.step[2];
            // spectra are shared where they are those of the same values: nothing writes the buffer in between
            if (!written_between(P, L.w, std::min(fwd, bwd), std::max(fwd, bwd))) L.spectra = hold_spectra(l, plan_kernel_bytes(&L.plan));
            if (grad > fwd && grad > bwd && !written_between(P, L.in, fwd, grad) && !written_between(P, L.gout, bwd, grad))
                L.memo = hold_spectra(l, plan_memo_bytes(&L.plan));
            // On one stream, products and inverse transforms of a small layer's gradient share the launches of those of the backward pass, if no
            // operation could tell: 2D net, a round of 48 -> 40 launches, 387 -> 344 us.
            if (L.memo != kNone && L.spectra != kNone && P.streams == 1 && bwd > fwd && plan_joins_gradient(&L.plan) &&
                !touched_between(P, P.steps[grad].op.buf[2], bwd - 1, grad)) {
                L.joined = true;
                P.steps[grad].skip = true;
            }
        }
    }
    // It completes a gradient that nothing touches between the operation that makes it and the update; those of biases
    // are summed in one launch before it where nothing writes their operands later, each in its place otherwise
    P.completes.assign(P.update_steps.size(), -1);
    for (size_t u = 0; u < P.update_steps.size(); ++u) {
        const int at_update = P.update_steps[u], g = P.steps[at_update].op.buf[0];
        for (int i = 0; i < at_update; ++i) {
            Step& s = P.steps[i];
            if (s.kind == ZNN_OP_BIAS_GRAD && s.op.buf[1] == g) {
                if (touched_between(P, g, i, at_update)) continue;
                s.own = take(sizeof(float) * s.op.maps * bias_spans(s.op));
                P.completes[u] = i;
                if (last_write[s.op.buf[0]] > i) continue;
                s.skip = true;
                P.bias_steps.push_back(i);
            } else if (s.kind == ZNN_OP_CONV_WGRAD && s.op.buf[2] == g) {
                const Layer& L = P.layers[s.layer];
                if (L.plan.mode != ZNN_DIRECT || touched_between(P, g, i, at_update)) continue;
                s.own = hold(s.layer, grad_sums_bytes(L.plan.g));
                if (s.own != kNone) P.completes[u] = i;
            }
        }
    }
    // On one stream the kernel gradients of small layers, which nothing waits for, go to the end, where one launch copies the
    // images of all, if nothing writes their operands later; on several they run beside the passes.
    std::vector<int> joins;
    for (int i = 0; i < n && P.streams == 1; ++i) {
        Step& s = P.steps[i];
        if (s.kind != ZNN_OP_CONV_WGRAD || s.own == kNone || last_write[s.op.buf[0]] >= i || last_write[s.op.buf[1]] >= i) continue;
        const Geom& g = P.layers[s.layer].plan.g;
        if (grad_joins(g)) joins.push_back(i);
        // As one launch with the sums of the biases: a gradient of few or small maps leaves most of the chip idle.  Six-layer 3D net, three of 7, 21 and 9 us
        // and 5 of the biases: a round 284 -> 268 us; 2D net 344 -> 332; sparse net, two of 7 and 19 us, 630 -> 618.
        else if (grad_is_few(g)) {
            s.skip = true;
            P.few_steps.push_back(i);
        }
    }
    for (int i : joins) {
        Step& s = P.steps[i];
        if (joins.size() > 1) s.copies = hold(s.layer, grad_copies_bytes(P.layers[s.layer].plan.g));
        if (s.copies == kNone) continue;
        s.skip = true;
        P.grad_steps.push_back(i);
    }
    add(STEP_FEW).skip = P.few_steps.empty();
    add(STEP_GRADS).skip = P.grad_steps.empty();
    add(STEP_BIAS).skip = P.bias_steps.empty() || !P.few_steps.empty();
    add(STEP_UPDATE).skip = P.update_steps.empty();
    // scratch of the passes: one area per stream
    std::vector<size_t> need(P.streams, 0);
    for (Step& s : P.steps) {
        if (s.layer < 0 || s.copies != kNone || (s.kind == ZNN_OP_CONV_WGRAD && P.layers[s.layer].joined)) continue;
        const Layer& L = P.layers[s.layer];
        const Geom& g = L.plan.g;
        if (s.kind == ZNN_OP_CONV_WGRAD) s.pass_bytes = s.own != kNone ? grad_copies_bytes(g) : plan_pass_bytes(&L.plan, s.kind, false);
        else if (L.packed[s.kind] != kNone) {
            const int splits = conv_splits(g, s.kind == ZNN_OP_CONV_BWD);
            s.pass_bytes = splits > 1 ? sizeof(float) * splits * (s.kind ? (size_t)g.f * g.nvol() : (size_t)g.fo * g.ovol()) : 0;
        } else s.pass_bytes = plan_pass_bytes(&L.plan, L.joined && s.kind == ZNN_OP_CONV_BWD ? ZNN_PASS_WGRAD : s.kind, L.spectra != kNone);
        need[s.stream] = std::max(need[s.stream], align256(s.pass_bytes));
    }
    P.area.resize(P.streams);
    for (int t = 0; t < P.streams; ++t) P.area[t] = take(need[t]);
    P.scratch = at;
    return ZNN_OK;
}

// whether a pass of a layer with shared kernel spectra is the one that makes them
bool transforms_kernels(const Layer& L, int kind) { return L.step[kind] < L.step[1 - kind]; }

// What every step reads and writes: buffers, the sums that steps leave for the update, what the passes of a layer share.
void name_resources(znn_program& P, int& resources)
{
    const int own = P.buffers, shared = own + (int)P.steps.size();      // shared: two per layer
    resources = shared + 2 * (int)P.layers.size();
    for (size_t i = 0; i < P.steps.size(); ++i) {
        Step& s = P.steps[i];
        const int* b = s.op.buf;
        auto rd = [&](int x) { if (x >= 0) s.reads.push_back(x); };
        auto wr = [&](int x) { if (x >= 0) s.writes.push_back(x); };
        if (s.kind == STEP_PACK) {
            for (size_t l = 0; l < P.layers.size(); ++l) {
                const Layer& L = P.layers[l];
                if (L.packed[0] != kNone || L.packed[1] != kNone) { rd(L.w); wr(shared + 2 * (int)l); }
            }
        } else if (s.kind == STEP_GRADS) {
            for (int q : P.grad_steps) { rd(P.steps[q].op.buf[0]); rd(P.steps[q].op.buf[1]); wr(own + q); }
        } else if (s.kind == STEP_FEW) {
            for (int q : P.few_steps) { rd(P.steps[q].op.buf[0]); rd(P.steps[q].op.buf[1]); wr(own + q); }
            for (int q : P.bias_steps) { rd(P.steps[q].op.buf[0]); wr(own + q); }
        } else if (s.kind == STEP_BIAS) {
            for (int q : P.bias_steps) { rd(P.steps[q].op.buf[0]); wr(own + q); }
        } else if (s.kind == STEP_UPDATE) {
            for (size_t u = 0; u < P.update_steps.size(); ++u) {
                const znn_op& o = P.steps[P.update_steps[u]].op;
                if (P.completes[u] >= 0) { rd(own + P.completes[u]); wr(o.buf[0]); }
                else rd(o.buf[0]);
                wr(o.buf[1]);
            }
        } else if (s.skip) continue;
        else switch (s.kind) {
            case ZNN_OP_CONV_FWD: case ZNN_OP_CONV_BWD: {
                const Layer& L = P.layers[s.layer];
                const int kernels = shared + 2 * s.layer, nodes = kernels + 1;
                rd(b[0]);
                if (L.packed[s.kind] != kNone || (L.spectra != kNone && !transforms_kernels(L, s.kind))) rd(kernels);
                else { rd(b[1]); if (L.spectra != kNone) wr(kernels); }
                if (L.memo != kNone) wr(nodes);
                if (L.joined && s.kind == ZNN_OP_CONV_BWD) wr(P.steps[L.step[2]].op.buf[2]);
                wr(b[2]);
                rd(b[3]);
                wr(b[4]);
                break;
            }
            case ZNN_OP_CONV_WGRAD:
                rd(b[0]); rd(b[1]);
                if (P.layers[s.layer].memo != kNone) rd(shared + 2 * s.layer + 1);
                wr(s.own != kNone ? own + (int)i : b[2]);
                break;
            default:
                for (int q = 0; q < 8; ++q) {
                    if (kForm[s.kind].reads >> q & 1) rd(b[q]);
                    if (kForm[s.kind].writes >> q & 1) wr(s.own != kNone ? own + (int)i : b[q]);
                }
        }
    }
}

// Waits between streams, without those that follow from earlier ones.
int place_waits(znn_program& P)
{
    int resources = 0;
    name_resources(P, resources);
    const int n = (int)P.steps.size(), S = P.streams;
    std::vector<int> writer(resources, -1), last(S, -1);
    std::vector<std::vector<int>> readers(resources), after(n);
    std::vector<std::vector<int>> over(S, std::vector<int>(S, -1));     // over[s][t]: last step of stream t over before stream s goes on
    std::vector<char> record(n, 0);
    P.used.assign(S, 0);
    for (int i = 0; i < n; ++i) {
        Step& s = P.steps[i];
        if (s.skip) continue;
        P.used[s.stream] = 1;
        std::vector<int> deps;
        for (int r : s.reads) if (writer[r] >= 0) deps.push_back(writer[r]);
        for (int w : s.writes) {
            if (writer[w] >= 0) deps.push_back(writer[w]);
            deps.insert(deps.end(), readers[w].begin(), readers[w].end());
        }
        std::sort(deps.begin(), deps.end());
        for (size_t k = deps.size(); k-- > 0;) {
            const int d = deps[k], t = P.steps[d].stream;
            if (t == s.stream || over[s.stream][t] >= d) continue;
            s.waits.push_back(d);
            record[d] = 1;
            for (int q = 0; q < S; ++q) over[s.stream][q] = std::max(over[s.stream][q], after[d][q]);
        }
        for (int r : s.reads) readers[r].push_back(i);
        for (int w : s.writes) { writer[w] = i; readers[w].clear(); }
        over[s.stream][s.stream] = i;
        after[i] = over[s.stream];
        last[s.stream] = i;
    }
    for (int t = 1; t < S; ++t)
        if (last[t] >= 0 && over[0][t] < last[t]) { record[last[t]] = 1; P.last_waits.push_back(last[t]); }
    for (int i = 0; i < n; ++i)
        if (record[i] && hipEventCreateWithFlags(&P.steps[i].event, hipEventDisableTiming) != hipSuccess)
            return fail(ZNN_EHIP, "cannot create an event");
    bool side = false;
    for (int t = 1; t < S; ++t) side = side || P.used[t];
    if (side && hipEventCreateWithFlags(&P.start, hipEventDisableTiming) != hipSuccess)
        return fail(ZNN_EHIP, "cannot create an event");
    return ZNN_OK;
}

// ---------------------------------------------------------------- launches
unsigned blocks_of(long count) { return (unsigned)((count + 255) / 256); }

int run_pack(const znn_program& P, float* const* buf, char* scratch, hipStream_t s)
{
    std::vector<PackItem> items;
    for (const Layer& L : P.layers)
        for (int b = 0; b < 2; ++b)
            if (L.packed[b] != kNone)
                items.push_back(conv_pack_item(L.plan.g, b == 1, buf[L.w], scratch + L.packed[b]));
    return conv_pack_weights(items.data(), (int)items.size(), s);
}

BiasItem bias_item(const Step& b, float* const* buf, char* scratch, unsigned first)
{
    return BiasItem{buf[b.op.buf[0]], (float*)(scratch + b.own), voxels(b.op), bias_spans(b.op), first};
}

int run_bias(const znn_program& P, const std::vector<int>& steps, float* const* buf, char* scratch, hipStream_t s)
{
    for (size_t i0 = 0; i0 < steps.size(); i0 += kBiasItems) {
        BiasArgs A = {};
        unsigned blocks = 0;
        for (; A.n < kBiasItems && i0 + A.n < steps.size(); ++A.n) {
            const Step& b = P.steps[steps[i0 + A.n]];
            A.item[A.n] = bias_item(b, buf, scratch, blocks);
            blocks += (unsigned)bias_spans(b.op) * b.op.maps;
        }
        ZNN_LAUNCH("bias gradients", s, k_bias_parts, dim3(blocks), dim3(256), 0, A);
    }
    return check_launch("bias gradients");
}

int run_grads(znn_program& P, float* const* buf, char* scratch, hipStream_t s)
{
    std::vector<GradItem> items;
    for (int q : P.grad_steps) {
        Step& t = P.steps[q];
        items.push_back(GradItem{&P.layers[t.layer].plan.g, buf[t.op.buf[0]], buf[t.op.buf[1]], (float*)(scratch + t.own),
                                 scratch + t.copies, &t.sum});
    }
    return grads_partial(items.data(), (int)items.size(), s);
}

int run_few(znn_program& P, float* const* buf, char* scratch, hipStream_t s)
{
    std::vector<GradItem> items;
    std::vector<BiasItem> bias;
    for (int q : P.few_steps) {
        Step& t = P.steps[q];
        items.push_back(GradItem{&P.layers[t.layer].plan.g, buf[t.op.buf[0]], buf[t.op.buf[1]], (float*)(scratch + t.own), nullptr, &t.sum});
    }
    size_t blocks = 0;
    for (int q : P.bias_steps) {
        bias.push_back(bias_item(P.steps[q], buf, scratch, (unsigned)blocks));
        blocks += (size_t)bias.back().spans * P.steps[q].op.maps;
    }
    // more biases than go with the gradients, in a launch of their own
    if (bias.size() > kFewBiases || blocks > kFewBiasGroups) {
        const int rc = run_bias(P, P.bias_steps, buf, scratch, s);
        if (rc != ZNN_OK) return rc;
        bias.clear();
        blocks = 0;
    }
    return few_grads(items.data(), (int)items.size(), bias.data(), (int)bias.size(), (unsigned)blocks, s);
}

int run_update(const znn_program& P, float* const* buf, char* scratch, float eta, hipStream_t s)
{
    for (size_t u = 0; u < P.update_steps.size();) {
        UpdateArgs A = {};
        A.eta = eta;
        unsigned blocks = 0;
        for (; A.n < kUpdateItems && u < P.update_steps.size(); ++A.n, ++u) {
            const Step& t = P.steps[P.update_steps[u]];
            const int done_by = P.completes[u];
            UpdateItem& I = A.item[A.n];
            I.grad = buf[t.op.buf[0]]; I.p = buf[t.op.buf[1]];
            I.first = blocks;
            I.total = elements(t.op);
            // layers that share parameters take their steps one after another
            bool shared = false;
            for (int q = 0; q < A.n && !shared; ++q) shared = I.p < A.item[q].p + A.item[q].total && A.item[q].p < I.p + I.total;
            if (shared) break;
            if (done_by >= 0) {
                const Step& d = P.steps[done_by];
                I.src = (const float*)(scratch + d.own);
                if (d.kind == ZNN_OP_BIAS_GRAD) { I.kind = 3; I.sum.ksplit = bias_spans(d.op); }
                else {
                    I.kind = d.sum.four ? 2 : 1;
                    I.sum = d.sum;
                }
            }
            blocks += I.kind == 2 ? (unsigned)((I.sum.slots + 63) / 64) : blocks_of(I.kind == 1 ? I.sum.slots : I.total);
        }
        ZNN_LAUNCH("gradient sums and update", s, k_update, dim3(blocks), dim3(256), 0, A);
    }
    return check_launch("gradient sums and update");
}

int run_conv(znn_program& P, Step& t, float* const* buf, char* scratch, hipStream_t s)
{
    Layer& L = P.layers[t.layer];
    const Geom& g = L.plan.g;
    const znn_op& o = t.op;
    const bool bwd = t.kind == ZNN_OP_CONV_BWD;
    char* const area = scratch + P.area[t.stream];
    auto at = [&](int q) -> float* { return o.buf[q] < 0 ? nullptr : buf[o.buf[q]]; };
    if (t.kind == ZNN_OP_CONV_WGRAD) {
        if (t.own != kNone) return grad_partial(g, at(0), at(1), (float*)(scratch + t.own), area, &t.sum, s);
        if (L.memo != kNone) return plan_wgrad_memo(&L.plan, (float2*)(scratch + L.memo), at(2), area, s);
        return plan_pass(&L.plan, ZNN_PASS_WGRAD, at(0), at(1), at(2), nullptr, area, nullptr, s);
    }
    const long count = bwd ? (long)g.f * g.nvol() : (long)g.fo * g.ovol();
    // what follows the sums: the next edge's transfer function, or the derivative of the one below
    Finish F = {};
    if (bwd) F.deriv = at(3); else { F.bias = at(3); F.y = at(4); }
    F.fn = o.fn;
    bool finished = !F.y && !F.deriv;
    // One buffer for out and y: a pass may write them in any order and reads its sums again where they are not finite, so y follows behind it.
    const Finish here = F.y == at(2) ? Finish{} : F;
    int rc;
    const bool few = L.plan.mode == ZNN_DIRECT && !conv_takes_packed(g, bwd);
    if (few || L.packed[bwd] != kNone) {
        const int splits = conv_splits(g, bwd);
        const bool inside = (here.y || here.deriv) && splits == 1 && o.fn == ZNN_RECTIFY;
        rc = conv_pass(g, bwd, at(0), at(1), few ? nullptr : scratch + L.packed[bwd], at(2), (float*)area, inside ? here : Finish{}, s);
        if (rc != ZNN_OK) return rc;
        if (splits > 1) {
            if (F.deriv) {
                ZNN_LAUNCH("sum of shares, derivative", s, k_finish_bwd, dim3(blocks_of(count)), dim3(256), 0, (const float*)area, F.deriv, at(2),
                           count, splits, o.fn);
                finished = true;
            } else if (here.y && g.fo <= 65535) {
                ZNN_LAUNCH("sum of shares, transfer", s, k_finish_fwd, dim3(blocks_of(g.ovol()), (unsigned)g.fo), dim3(256), 0,
                           (const float*)area, at(2), F.bias, F.y, (int)g.ovol(), count, splits, o.fn);
                finished = true;
            } else rc = conv_sum(g, bwd, (const float*)area, at(2), s);
            if (rc != ZNN_OK) return rc;
        } else finished = finished || inside;
    } else {
        float2* What = L.spectra != kNone ? (float2*)(scratch + L.spectra) : nullptr;
        float2* memo = L.memo != kNone ? (float2*)(scratch + L.memo) : nullptr;
        const bool held = What && !transforms_kernels(L, t.kind);
        PassMore more = {What, bwd && L.joined ? buf[P.steps[L.step[2]].op.buf[2]] : nullptr, here, false};
        rc = plan_pass(&L.plan, t.kind, at(0), held ? nullptr : at(1), at(2), held ? What : nullptr, area, memo, s, &more);
        if (rc != ZNN_OK) return rc;
        finished = finished || more.finished;
    }
    if (!finished) {
        if (F.y) return znn_transfer_fn_fwd(o.fn, g.fo, g.ovol(), at(2), F.bias, F.y, s);
        ZNN_LAUNCH("transfer derivative", s, k_derivative_in_place, dim3(blocks_of(count)), dim3(256), 0, at(2), F.deriv, count, o.fn);
    }
    return check_launch("convolution of a program");
}

int run_step(znn_program& P, Step& t, float* const* buf, char* scratch, float eta, hipStream_t s)
{
    const znn_op& o = t.op;
    auto at = [&](int q) -> float* { return o.buf[q] < 0 ? nullptr : buf[o.buf[q]]; };
    const long count = t.kind > ZNN_OP_CONV_WGRAD ? elements(o) : 0;
    switch (t.kind) {
        case STEP_PACK: return run_pack(P, buf, scratch, s);
        case STEP_GRADS: return run_grads(P, buf, scratch, s);
        case STEP_FEW: return run_few(P, buf, scratch, s);
        case STEP_BIAS: return run_bias(P, P.bias_steps, buf, scratch, s);
        case STEP_UPDATE: return run_update(P, buf, scratch, eta, s);
        case ZNN_OP_TRANSFER_FWD: return znn_transfer_fn_fwd(o.fn, o.maps, voxels(o), at(0), at(1), at(2), s);
        case ZNN_OP_TRANSFER_BWD: return znn_transfer_fn_bwd(o.fn, o.maps, voxels(o), at(0), at(1), at(2), s);
        case ZNN_OP_BIAS_GRAD:
            if (t.own != kNone) return run_bias(P, {(int)(&t - P.steps.data())}, buf, scratch, s);
            return znn_bias_grad(o.maps, voxels(o), at(0), at(1), s);
        case ZNN_OP_FILTER_FWD:
            return znn_maxfilter3d_sparse_fwd(o.maps, o.n, o.window, o.sparsity, at(0), at(1), (int32_t*)at(2), s);
        case ZNN_OP_FILTER_BWD:
            return maxfilter_bwd(o.maps, o.n, o.window, o.sparsity, at(0), (const int32_t*)at(1), at(2), at(3), o.fn, s);
        case ZNN_OP_POOL_FWD: return znn_maxpool3d_fwd(o.maps, o.n, o.window, at(0), at(1), (int32_t*)at(2), s);
        case ZNN_OP_POOL_BWD: {
            int rc = znn_maxpool3d_bwd(o.maps, o.n, o.window, at(0), (const int32_t*)at(1), at(2), s);
            if (rc != ZNN_OK || o.buf[3] < 0) return rc;
            ZNN_LAUNCH("transfer derivative", s, k_derivative_in_place, dim3(blocks_of(count)), dim3(256), 0, at(2), at(3), count, o.fn);
            return check_launch("transfer derivative");
        }
        case ZNN_OP_LOSS_GRAD:
            ZNN_LAUNCH("loss gradient", s, k_loss_finish, dim3(blocks_of(count)), dim3(256), 0, count, at(0), at(1), at(2), at(3), o.loss, o.fn);
            return check_launch("loss gradient");
        case ZNN_OP_UPDATE: return znn_sgd_update(count, eta, at(0), at(1), s);
        case ZNN_OP_NODE_SUM: {
            SumArgs A = {};
            for (int q = 1; q < 7 && o.buf[q] >= 0; ++q) A.part[A.parts++] = at(q);
            A.y = at(7); A.out = at(0); A.count = count; A.fn = o.fn;
            ZNN_LAUNCH("node sum", s, k_node_sum, dim3(blocks_of(count)), dim3(256), 0, A);
            return check_launch("node sum");
        }
    }
    return run_conv(P, t, buf, scratch, s);
}

}  // namespace

}  // namespace znn

extern "C" {

int znn_program_create(const znn_op* ops, int32_t count, int32_t buffers, int32_t streams, znn_program** program)
{
    if (!ops || !program) return fail(ZNN_EINVAL, "NULL argument");
    if (count < 1 || buffers < 1 || streams < 1) return fail(ZNN_EINVAL, "a program needs operations, buffers and a stream");
    znn_program* P = new (std::nothrow) znn_program;
    if (!P) return fail(ZNN_EINVAL, "out of host memory");
    P->buffers = buffers; P->streams = streams; P->start = nullptr; P->scratch = 0;
    int rc;
    try {
        rc = place_steps(*P, ops, count);
        if (rc == ZNN_OK) rc = place_waits(*P);
    } catch (const std::bad_alloc&) {       // callers are in other languages: no exception leaves the library
        rc = fail(ZNN_EINVAL, "out of host memory");
    }
    if (rc != ZNN_OK) { znn_program_destroy(P); return rc; }
    *program = P;
    return ZNN_OK;
}

void znn_program_destroy(znn_program* program)
{
    if (!program) return;
    for (Step& s : program->steps) if (s.event) (void)hipEventDestroy(s.event);
    if (program->start) (void)hipEventDestroy(program->start);
    delete program;
}

int znn_program_scratch_bytes(const znn_program* program, size_t* bytes)
{
    if (!program || !bytes) return fail(ZNN_EINVAL, "NULL argument");
    *bytes = program->scratch;
    return ZNN_OK;
}

int znn_program_run(znn_program* program, void* const* buffers, void* scratch, size_t scratch_bytes, float eta,
                    void* const* streams)
{
    if (!program || !buffers || !streams) return fail(ZNN_EINVAL, "NULL argument");
    znn_program& P = *program;
    for (int b = 0; b < P.buffers; ++b) if (!buffers[b]) return fail(ZNN_EINVAL, "buffer %d is NULL", b);
    if (P.scratch) {
        if (!scratch) return fail(ZNN_EWORKSPACE, "scratch is NULL but %zu bytes are needed", P.scratch);
        if ((uintptr_t)scratch & 255) return fail(ZNN_EWORKSPACE, "scratch is not 256-byte aligned");
        if (scratch_bytes < P.scratch) return fail(ZNN_EWORKSPACE, "scratch has %zu bytes, %zu needed", scratch_bytes, P.scratch);
    }
    hipStream_t const* st = (hipStream_t const*)streams;
    bool ok = true;
    if (P.start) {
        ok = hipEventRecord(P.start, st[0]) == hipSuccess;
        for (int t = 1; t < P.streams; ++t) if (P.used[t]) ok = ok && hipStreamWaitEvent(st[t], P.start, 0) == hipSuccess;
    }
    // a failed launch still leaves the side streams joined below
    int rc = ZNN_OK;
    for (Step& s : P.steps) {
        if (s.skip) continue;
        for (int d : s.waits) ok = ok && hipStreamWaitEvent(st[s.stream], P.steps[d].event, 0) == hipSuccess;
        try {
            if (rc == ZNN_OK) rc = run_step(P, s, (float* const*)buffers, (char*)scratch, eta, st[s.stream]);
        } catch (const std::bad_alloc&) {
            rc = fail(ZNN_EINVAL, "out of host memory");
        }
        if (s.event) ok = ok && hipEventRecord(s.event, st[s.stream]) == hipSuccess;
    }
    for (int d : P.last_waits) ok = ok && hipStreamWaitEvent(st[0], P.steps[d].event, 0) == hipSuccess;
    if (rc != ZNN_OK) return rc;
    return ok ? ZNN_OK : fail(ZNN_EHIP, "cannot order the streams of the program");
}

}  // extern "C"
