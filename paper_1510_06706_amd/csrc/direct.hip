// Direct method: which kernels take a pass, and the pass in pieces for rounds that finish several layers in one launch.
//
// Forward and backward pass: the kernel on split operands (direct_split_impl.h) or the one on the vector ALUs (direct_few.hip),
// whichever is expected to be faster, preparation and the sum of the shares included: the former packs its weights in a launch of
// its own and pads the input-side maps to eight.  The backward pass is the forward one with the roles of the two node sets
// swapped, the kernel reflected and the output gradient zero-extended by s (k - 1) on every side (Section 3.1).  The kernel
// gradient likewise: the split kernel copies both images first.
#include <algorithm>

#include "direct.h"

namespace znn {

namespace {

// x = sum of the shares in ascending order
__global__ void __launch_bounds__(256)
k_conv_reduce(const float* __restrict__ partial, float* __restrict__ dst, long count, int splits)
{
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    if (t >= count) return;
    float acc = partial[t];
    for (int s = 1; s < splits; ++s) acc += partial[(long)s * count + t];
    dst[t] = acc;
}

long result_count(const Geom& g, bool backward) { return backward ? (long)g.f * g.nvol() : (long)g.fo * g.ovol(); }

// ok = false: the vector ALUs take the pass
SplitChoice way(const Geom& g, bool backward)
{
    SplitChoice c = choose_split(g, backward);
    if (c.ok && few_conv_seconds(g, backward) < split_seconds(c) + 3e-6) c.ok = false;
    return c;
}

bool few_gradient(const Geom& g) { return !split_grad_supported(g) || few_grad_seconds(g) < split_grad_seconds(g); }

}  // namespace

bool conv_takes_packed(const Geom& g, bool backward) { return way(g, backward).ok; }

double conv_seconds(const Geom& g, bool backward)
{
    const SplitChoice c = way(g, backward);
    return c.ok ? split_seconds(c) : few_conv_seconds(g, backward);
}

size_t conv_packed_bytes(const Geom& g, bool backward)
{
    const SplitChoice c = way(g, backward);
    return c.ok ? split_packed_bytes(c) : 0;
}

PackItem conv_pack_item(const Geom& g, bool backward, const float* w, void* wp)
{
    return split_pack_item(g, choose_split(g, backward), backward, w, wp);
}

int conv_pack_weights(const PackItem* items, int n, hipStream_t s) { return split_pack_weights(items, n, s); }

int conv_splits(const Geom& g, bool backward)
{
    const SplitChoice c = way(g, backward);
    return c.ok ? c.splits : 1;
}

// With more than one share of the input maps (conv_splits) the sums go to `partial`, one array of result maps per share, and the
// caller adds them in ascending order.
int conv_pass(const Geom& g, bool backward, const float* src, const float* w, const void* wp, float* dst, float* partial,
              const Finish& finish, hipStream_t s)
{
    const SplitChoice c = way(g, backward);
    return c.ok ? split_conv(g, c, backward, src, w, wp, dst, partial, finish, s) : few_conv(g, backward, src, w, dst, finish, s);
}

int conv_sum(const Geom& g, bool backward, const float* partial, float* dst, hipStream_t s)
{
    const long count = result_count(g, backward);
    ZNN_LAUNCH("sum over input-map shares", s, k_conv_reduce, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, partial, dst, count,
               conv_splits(g, backward));
    return check_launch("sum over input-map shares");
}

double grad_seconds(const Geom& g) { return few_gradient(g) ? few_grad_seconds(g) : split_grad_seconds(g); }
size_t grad_sums_bytes(const Geom& g) { return few_gradient(g) ? few_grad_sums_bytes(g) : split_grad_sums_bytes(g); }
size_t grad_copies_bytes(const Geom& g) { return few_gradient(g) ? 0 : split_grad_copies_bytes(g); }

int grad_partial(const Geom& g, const float* in, const float* gout, float* partial, void* copies, WgradSum* sum, hipStream_t s)
{
    return few_gradient(g) ? few_grad(g, in, gout, partial, nullptr, sum, s)
                           : split_grad(g, GradItem{&g, in, gout, partial, copies, sum}, s);
}

bool grad_joins(const Geom& g) { return !few_gradient(g) && split_grad_joins(g); }
int grads_partial(const GradItem* items, int count, hipStream_t s) { return split_grads(items, count, s); }

static size_t conv_workspace(const Geom& g, bool backward)
{
    const int splits = conv_splits(g, backward);
    return conv_packed_bytes(g, backward) + (splits > 1 ? align256((size_t)splits * result_count(g, backward) * sizeof(float)) : 0);
}

size_t direct_workspace_bytes(const Geom& g, int pass)
{
    if (pass != ZNN_PASS_WGRAD) return conv_workspace(g, pass == ZNN_PASS_BWD);
    return grad_sums_bytes(g) + grad_copies_bytes(g);
}

static int direct_conv(const Geom& g, bool backward, const float* src, const float* w, float* dst, void* ws, hipStream_t s)
{
    float* partial = (float*)((char*)ws + conv_packed_bytes(g, backward));
    int rc = ZNN_OK;
    if (conv_takes_packed(g, backward)) {
        const PackItem p = conv_pack_item(g, backward, w, ws);
        rc = conv_pack_weights(&p, 1, s);
    }
    if (rc == ZNN_OK) rc = conv_pass(g, backward, src, w, ws, dst, partial, Finish{}, s);
    if (rc != ZNN_OK || conv_splits(g, backward) == 1) return rc;
    return conv_sum(g, backward, partial, dst, s);
}

int direct_fwd(const Geom& g, const float* in, const float* w, float* out, void* ws, hipStream_t s)
{
    return direct_conv(g, false, in, w, out, ws, s);
}

// The forward pass one group of output maps after another (the maps that a workgroup takes): weights and sums of one at a time, the
// same launches otherwise.  For callers whose scratch does not hold those of all.
static Geom group_of(const Geom& g, const SplitChoice& c, int first)
{
    Geom q = g;
    q.fo = std::min(16 * c.NJ, g.fo - first);
    return q;
}

static size_t group_bytes(const Geom& g, const SplitChoice& c)
{
    const size_t sums = c.splits > 1 ? align256(sizeof(float) * c.splits * result_count(group_of(g, c, 0), false)) : 0;
    return split_packed_bytes(c) + sums;
}

size_t direct_fwd_least(const Geom& g)
{
    SplitChoice c = way(g, false);
    if (!c.ok) return 0;
    c.jgroups = 1;
    const size_t bytes = group_bytes(g, c);
    return bytes > ZNN_STATIC_SCRATCH_BYTES ? 0 : std::min(conv_workspace(g, false), bytes);
}

int direct_fwd_groups(const Geom& g, const float* in, const float* w, float* out, void* ws, hipStream_t s)
{
    SplitChoice c = way(g, false);
    c.jgroups = 1;
    if (!c.ok || group_bytes(g, c) > ZNN_STATIC_SCRATCH_BYTES) return few_conv(g, false, in, w, out, Finish{}, s);
    float* partial = (float*)((char*)ws + split_packed_bytes(c));
    for (int first = 0; first < g.fo; first += 16 * c.NJ) {
        const Geom q = group_of(g, c, first);
        float* dst = out + (long)first * g.ovol();
        const float* wq = w + (long)first * g.f * g.kvol();
        const PackItem p = split_pack_item(q, c, false, wq, ws);
        int rc = split_pack_weights(&p, 1, s);
        if (rc == ZNN_OK) rc = split_conv(q, c, false, in, wq, ws, dst, partial, Finish{}, s);
        if (rc != ZNN_OK) return rc;
        if (c.splits == 1) continue;
        const long count = result_count(q, false);
        ZNN_LAUNCH("sum over input-map shares", s, k_conv_reduce, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, partial, dst, count,
                   c.splits);
    }
    return check_launch("direct forward in groups of maps");
}

int direct_bwd(const Geom& g, const float* gout, const float* w, float* gin, void* ws, hipStream_t s)
{
    return direct_conv(g, true, gout, w, gin, ws, s);
}

int direct_wgrad(const Geom& g, const float* in, const float* gout, float* gw, void* ws, hipStream_t s)
{
    WgradSum S;
    if (few_gradient(g) && few_grad_shares(g) == 1) return few_grad(g, in, gout, nullptr, gw, &S, s);
    const int rc = grad_partial(g, in, gout, (float*)ws, (char*)ws + grad_sums_bytes(g), &S, s);
    return rc == ZNN_OK ? sum_shares(S, (const float*)ws, gw, s) : rc;
}

}  // namespace znn
