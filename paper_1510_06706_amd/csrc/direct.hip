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

// x = sum of the shares in ascending order, behind what x holds where `more`
__global__ void __launch_bounds__(256)
k_conv_reduce(const float* __restrict__ partial, float* __restrict__ dst, long count, int splits, int more)
{
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    if (t >= count) return;
    float acc = partial[t];
    if (more) acc = dst[t] + acc;       // uniform
    for (int s = 1; s < splits; ++s) acc += partial[(long)s * count + t];
    dst[t] = acc;
}

void reduce(const float* partial, float* dst, long count, int splits, bool more, hipStream_t s)
{
    ZNN_LAUNCH("sum over input-map shares", s, k_conv_reduce, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, partial, dst, count, splits,
               more ? 1 : 0);
}

long result_count(const Geom& g, bool backward) { return backward ? (long)g.f * g.nvol() : (long)g.fo * g.ovol(); }

// ok = false: the vector ALUs take the pass.  Held against the price of waves that stage in between, which that of the vector ALUs was fitted beside, also where others
// stage; so what the vector ALUs took they take.
SplitChoice way(const Geom& g, bool backward)
{
    SplitChoice c = choose_split(g, backward);
    if (c.ok && few_conv_seconds(g, backward) < split_seconds(c.between) + 3e-6) c.ok = false;
    return c;
}

bool few_gradient(const Geom& g) { return !split_grad_supported(g) || few_grad_seconds(g) < split_grad_seconds(g); }

}  // namespace

bool conv_takes_packed(const Geom& g, bool backward) { return way(g, backward).ok; }

double conv_seconds(const Geom& g, bool backward)
{
    const SplitChoice c = way(g, backward);
    return c.ok ? split_seconds(c.between) : few_conv_seconds(g, backward);         // as the choice between the methods was fitted to (api.hip)
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
    reduce(partial, dst, result_count(g, backward), conv_splits(g, backward), false, s);
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

bool grad_is_few(const Geom& g) { return few_gradient(g); }
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

// The forward pass in the built-in scratch array: one group of output maps after another, and where the sums of all shares do not
// fit, a few shares after another.  Chunks, shares and the order of every sum are those of the ordinary call, so results are too, but
// where the sums of one share do not fit.
static Geom group_of(const Geom& g, const SplitChoice& c, int first)
{
    Geom q = g;
    q.fo = std::min(16 * c.NJ, g.fo - first);
    return q;
}

static size_t share_bytes(const Geom& g, const SplitChoice& c) { return sizeof(float) * result_count(group_of(g, c, 0), false); }

// c.jgroups = 1 and the largest groups whose weights and sums fit, or else the smallest; shares: those of a launch.  Not ok: the weights
// of sixteen output maps do not fit, and the vector ALUs take the pass.
static SplitChoice choose_groups(const Geom& g, int& shares)
{
    SplitChoice c = way(g, false);
    if (!c.ok) return c;
    const int tiles = (g.fo + 15) / 16;
    int groups = (tiles + c.NJ - 1) / c.NJ;
    c.jgroups = 1;
    for (; ; ++groups, c.NJ = (tiles + groups - 1) / groups) {
        const size_t packed = split_packed_bytes(c);
        c.ok = packed <= ZNN_STATIC_SCRATCH_BYTES;
        shares = c.ok && c.splits > 1 ? (int)std::min<size_t>(c.splits, (ZNN_STATIC_SCRATCH_BYTES - packed) / share_bytes(g, c)) : 1;
        if (c.NJ == 1 || (c.ok && shares == c.splits)) break;
    }
    // not even the sums of one share: one after another in the accumulators
    if (shares == 0) {
        shares = c.splits = 1;
        c.cps = c.nchunk;
    }
    c.ok = c.ok && split_place(c);
    return c;
}

// never more than the array holds
size_t direct_fwd_least(const Geom& g)
{
    int shares;
    const SplitChoice c = choose_groups(g, shares);
    if (!c.ok) return 0;
    return std::min(conv_workspace(g, false), split_packed_bytes(c) + (c.splits > 1 ? shares * share_bytes(g, c) : 0));
}

int direct_fwd_groups(const Geom& g, const float* in, const float* w, float* out, void* ws, hipStream_t s)
{
    int shares;
    const SplitChoice c = choose_groups(g, shares);
    if (!c.ok) return few_conv(g, false, in, w, out, Finish{}, s);
    float* partial = (float*)((char*)ws + split_packed_bytes(c));
    for (int first = 0; first < g.fo; first += 16 * c.NJ) {
        const Geom q = group_of(g, c, first);
        float* dst = out + (long)first * g.ovol();
        const float* wq = w + (long)first * g.f * g.kvol();
        const PackItem p = split_pack_item(q, c, false, wq, ws);
        int rc = split_pack_weights(&p, 1, s);
        for (int share = 0; share < c.splits && rc == ZNN_OK; share += shares) {
            const int n = std::min(shares, c.splits - share);
            // a share on its own goes where it belongs if it is the first, the others behind it
            rc = split_conv(q, c, false, in, wq, ws, n > 1 || share == 0 ? dst : partial, partial, Finish{}, s, share, n);
            if (rc == ZNN_OK && (n > 1 || share > 0)) reduce(partial, dst, result_count(q, false), n, share > 0, s);
        }
        if (rc != ZNN_OK) return rc;
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
