"""The direct kernels on operands split into three bf16 parts: edges of their tiles, sublattices of sparse
taps, shares of the input maps, and operands that are not finite.

The bound is derived, element by element, from S = sum of |products| (the oracle on absolute values): what the split leaves
out of a product is below 2^-24 of it, a step of 32 products is summed by six instructions, and then one fp32 addition per
step and share rounds a partial sum that is at most S.
"""
import numpy as np
import pytest

import oracle
from paper_1510_06706_amd import binding as znn
from paper_1510_06706_amd import synth
from direct_layers import BESIDE

pytestmark = pytest.mark.gpu

SHAPES = [
    # f, fo, n, k, s: map counts around the chunks of 8 and the tiles of 16, taps around the steps of 4
    (5, 1, (6, 7, 8), (1, 1, 1), (1, 1, 1)),            # one tap
    (8, 16, (9, 8, 17), (1, 2, 2), (1, 1, 1)),          # one full step
    (9, 17, (7, 9, 16), (1, 1, 5), (1, 1, 1)),          # a step and a tap
    (40, 40, (14, 13, 12), (3, 3, 3), (1, 1, 1)),
    (24, 81, (5, 20, 19), (2, 3, 4), (1, 1, 1)),        # two groups of map tiles
    (130, 7, (6, 6, 9), (2, 2, 2), (1, 1, 1)),          # many chunks, shares of them
    (6, 33, (1, 40, 23), (1, 7, 3), (1, 1, 1)),         # 2D
    (16, 8, (33, 4, 40), (3, 1, 3), (1, 1, 1)),
    (12, 12, (15, 14, 13), (3, 3, 3), (2, 3, 4)),       # sublattices of different extents
    (10, 10, (9, 9, 11), (3, 3, 3), (4, 4, 5)),         # result extents below the tap spacing
    (8, 24, (3, 30, 30), (1, 3, 3), (3, 2, 2)),         # spacing on an axis of one tap
    (48, 64, (20, 20, 20), (3, 3, 3), (1, 1, 1)),
    (72, 72, (10, 11, 12), (5, 4, 3), (1, 1, 1)),       # five map tiles
    (5, 5, (30, 9, 10), (17, 9, 7), (1, 1, 1)),         # 1071 taps
]


# Layers as small as some of those above take the kernels on the vector ALUs; these are the same edges on layers that do not, which
# the tests assert.
WIDE_SHAPES = [
    (64, 64, (32, 48, 48), (1, 1, 1), (1, 1, 1)),       # one tap
    (24, 40, (33, 34, 66), (1, 2, 2), (1, 1, 1)),       # one full step
    (17, 33, (44, 45, 46), (1, 1, 5), (1, 1, 1)),       # a step and a tap
    (130, 7, (26, 26, 29), (2, 2, 2), (1, 1, 1)),       # many chunks
    (40, 40, (25, 24, 23), (3, 3, 3), (2, 3, 4)),       # sublattices of different extents
    (64, 64, (25, 24, 31), (3, 3, 3), (8, 8, 9)),       # result extents around the tap spacing
]


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a.astype(np.float32))).to("cuda:0")


def tensors(f, fo, n, k, s, seed):
    x, w, g = synth.layer_tensors(synth.LayerShape("t", f, fo, n, k, 1.0, seed, s))
    return x, w, g


def kernels_of(call, *names):
    """The call's result; `names` are among the kernels that it launches."""
    import torch
    znn.trace_enable(True)
    try:
        result = call()
        torch.cuda.synchronize()
        launched = {name for name, _ in znn.trace_collect(64)}
    finally:
        znn.trace_enable(False)
    assert set(names) <= launched, (names, launched)
    return result


def bound(ref_abs, maps, taps):
    adds = -(-maps // 8) * -(-taps // 4) + -(-maps // 8)
    return (adds + 16) * 2.0 ** -24 * ref_abs


def passes_within_bound(f, fo, n, k, s, forward=(), backward=()):
    x, w, g = tensors(f, fo, n, k, s, 9100)
    taps = k[0] * k[1] * k[2]
    p = znn.Plan(f, fo, n, k, "direct", s)
    out = kernels_of(lambda: p.fwd(dev(x), dev(w)), *forward).cpu().numpy()
    gin = kernels_of(lambda: p.bwd(dev(g), dev(w)), *backward).cpu().numpy()
    err = np.abs(out.astype(np.float64) - oracle.conv3d_fwd(x, w, s))
    assert np.all(err <= bound(oracle.conv3d_fwd(np.abs(x), np.abs(w), s), f, taps))
    err = np.abs(gin.astype(np.float64) - oracle.conv3d_bwd(g, w, n, s))
    assert np.all(err <= bound(oracle.conv3d_bwd(np.abs(g), np.abs(w), n, s), fo, taps))
    p.close()


@pytest.mark.parametrize("f,fo,n,k,s", SHAPES)
def test_passes_stay_within_the_bound_of_the_split(f, fo, n, k, s):
    passes_within_bound(f, fo, n, k, s)


@pytest.mark.parametrize("f,fo,n,k,s", WIDE_SHAPES)
def test_passes_of_wide_layers_run_on_the_split_and_stay_within_its_bound(f, fo, n, k, s):
    passes_within_bound(f, fo, n, k, s, ["direct forward (MFMA)"], ["direct backward (MFMA)"])


@pytest.mark.parametrize("f,fo,n,k,s", [
    # layers whose halo boxes and weights other waves stage: one chunk and several, one and two map tiles in a group, odd and even steps
    (17, 31, (15, 15, 15), (3, 3, 3), (2, 2, 2)),       # sublattices, groups of maps forward
    (24, 24, (15, 15, 15), (3, 3, 3), (1, 1, 1)),       # a last map tile of eight
    (9, 33, (12, 11, 10), (3, 3, 3), (1, 1, 1)),        # chunks of eight maps and one, tiles of one
    (19, 23, (1, 46, 25), (1, 3, 3), (1, 1, 1)),        # two tiles a workgroup
    (7, 20, (20, 21, 22), (5, 2, 3), (1, 1, 1)),        # one chunk forward
    (13, 27, (14, 13, 15), (2, 3, 4), (1, 1, 1)),
    (7, 11, (15, 24, 41), (2, 6, 6), (1, 1, 1)),        # 18 steps
])
def test_passes_of_small_layers_run_on_the_split_within_its_bound_and_as_in_fp32(f, fo, n, k, s):
    passes_within_bound(f, fo, n, k, s, ["direct forward (MFMA)"], ["direct backward (MFMA)"])
    x, w, g = tensors(f, fo, n, k, s, 9110)
    p = znn.Plan(f, fo, n, k, "direct", s)
    out = p.fwd(dev(x), dev(w)).cpu().numpy()
    w[fo - 1], there = np.nan, np.arange(fo) == fo - 1              # a map of NaN stands alone
    got = p.fwd(dev(x), dev(w)).cpu().numpy()
    assert np.array_equal(got[~there], out[~there]) and np.all(np.isnan(got[there]))
    x[:, n[0] // 2, n[1] // 2, n[2] // 2], w[fo - 1] = np.inf, w[0]
    got, ref = p.fwd(dev(x), dev(w)).cpu().numpy(), oracle.conv3d_fwd(x, w, s)
    for kind in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(kind(got), kind(ref))
    p.close()


@pytest.mark.parametrize("f,fo,n,k,s,backward", [layer[:6] for layer in BESIDE])
def test_passes_that_stage_beside_stay_within_the_bound_and_as_in_fp32(f, fo, n, k, s, backward):
    s = (s, s, s)
    x, w, g = tensors(f, fo, n, k, s, 9111)
    p = znn.Plan(f, fo, n, k, "direct", s)
    src, of, maps = (g, w.swapaxes(0, 1), f) if backward else (x, w, fo)       # `of`: a view, weights by result map

    def run():
        return kernels_of(lambda: (p.bwd if backward else p.fwd)(dev(src), dev(w)), "direct backward (MFMA)" if backward else "direct forward (MFMA)").cpu().numpy()

    def exact(a, b):
        return oracle.conv3d_bwd(a, b, n, s) if backward else oracle.conv3d_fwd(a, b, s)

    out = run()
    assert np.all(np.abs(out.astype(np.float64) - exact(src, w)) <= bound(exact(np.abs(src), np.abs(w)), src.shape[0], k[0] * k[1] * k[2]))
    there = np.arange(maps) == maps - 1                             # a map of NaN stands alone
    kept = of[maps - 1].copy()
    of[maps - 1] = np.nan
    got = run()
    assert np.array_equal(got[~there], out[~there]) and np.all(np.isnan(got[there][np.isnan(exact(src, w)[there])]))
    of[maps - 1] = kept
    src[:, src.shape[1] // 2, src.shape[2] // 2, src.shape[3] // 2] = np.inf
    got, ref = run(), exact(src, w)
    for kind in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(kind(got), kind(ref))
    assert np.array_equal(got[np.isfinite(ref)], out[np.isfinite(ref)])
    p.close()


@pytest.mark.parametrize("n,s", [((26, 26, 26), (1, 1, 1)), ((34, 34, 34), (4, 4, 4))])
@pytest.mark.parametrize("half", [False, True])
def test_errors_of_the_split_have_no_common_sign(n, s, half):
    """The bf16 matrix instruction rounds sums downwards, by some 2^-28 of a step's sum; steps of alternating signs cancel it."""
    f, fo, k = 40, 40, (3, 3, 3)
    x, w, g = tensors(f, fo, n, k, s, 9106)
    if half:                                            # what a rectifier leaves
        x, g = np.maximum(x, 0), np.where(g > 0, g, 0).astype(np.float32)
    p = znn.Plan(f, fo, n, k, "direct", s)
    assert p.workspace_bytes(0) > 0 and p.workspace_bytes(1) > 0        # packed weights
    assert p.workspace_bytes(2) > 4 * (x.size + g.size)                 # copies of the images

    def unbiased(got, ref, steps):
        e, rms = got.cpu().numpy().astype(np.float64) - ref, np.sqrt(np.mean(ref ** 2))
        # four times the share of a step without a partner, and six standard deviations of the mean
        assert abs(np.mean(e)) <= rms * 2.0 ** -26 / np.sqrt(steps) + 6 * np.sqrt(np.mean(e ** 2) / e.size)

    unbiased(p.fwd(dev(x), dev(w)), oracle.conv3d_fwd(x, w, s), 35)
    unbiased(p.bwd(dev(g), dev(w)), oracle.conv3d_bwd(g, w, n, s), 35)
    unbiased(p.wgrad(dev(x), dev(g)), oracle.conv3d_wgrad(x, g, s), g[0].size // 32)
    p.close()


@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** 60])
def test_the_split_keeps_its_precision_at_any_scale(scale):
    f, fo, n, k, s = 16, 16, (10, 10, 10), (3, 3, 3), (1, 1, 1)
    x, w, g = tensors(f, fo, n, k, s, 9101)
    p = znn.Plan(f, fo, n, k, "direct", s)
    base, scaled = p.fwd(dev(x), dev(w)), p.fwd(dev(x * scale), dev(w / scale))
    assert np.array_equal(base.cpu().numpy(), scaled.cpu().numpy())
    p.close()


@pytest.mark.parametrize("ex,ew", [(-112, 0), (-120, 0), (-126, 0), (-138, 0), (0, -126), (-62, -62), (-66, -66), (45, 44)])
def test_the_split_keeps_its_precision_to_the_ends_of_the_range(ex, ew):
    """Operands near and below the smallest normal number, products near it, and sums that are finite only without the split's scale."""
    f, fo, n, k = 40, 40, (26, 26, 26), (3, 3, 3)
    x, w, g = tensors(f, fo, n, k, (1, 1, 1), 9108)
    p = znn.Plan(f, fo, n, k, "direct")
    assert p.workspace_bytes(0) > 0 and p.workspace_bytes(1) > 0        # packed weights
    assert p.workspace_bytes(2) > 4 * (x.size + g.size)                 # copies of the images
    x, g, v, w = (np.ldexp(a, e).astype(np.float32) for a, e in ((x, ex), (g, ex), (g, ew), (w, ew)))

    def close(got, ref, limit):
        # a share's sum and their sum may be subnormal: rounded to 2^-149
        assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= limit + 16 * 2.0 ** -149)

    def fp32(maps, ref_abs):        # sums taken again in fp32 round once per product
        return (27 * maps + 16) * 2.0 ** -24 * ref_abs if ex + ew > 80 else bound(ref_abs, maps, 27)

    close(p.fwd(dev(x), dev(w)), oracle.conv3d_fwd(x, w), fp32(f, oracle.conv3d_fwd(np.abs(x), np.abs(w))))
    close(p.bwd(dev(g), dev(w)), oracle.conv3d_bwd(g, w, n), fp32(fo, oracle.conv3d_bwd(np.abs(g), np.abs(w), n)))
    voxels = g[0].size
    close(p.wgrad(dev(x), dev(v)), oracle.conv3d_wgrad(x, v),
          (2 * (voxels // (1 if ex + ew > 80 else 32)) + 600) * 2.0 ** -24 * oracle.conv3d_wgrad(np.abs(x), np.abs(v)))
    p.close()


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
def test_operands_that_are_not_finite_act_as_in_fp32(value):
    f, fo, n, k, s = 9, 20, (11, 12, 13), (3, 3, 3), (1, 1, 1)
    x, w, g = tensors(f, fo, n, k, s, 9102)
    w *= 2.0 ** -10
    taps = 27
    p = znn.Plan(f, fo, n, k, "direct", s)

    def same(got, ref, limit):
        got = got.cpu().numpy().astype(np.float64)
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.array_equal(np.isneginf(got), np.isneginf(ref))
        ok = np.isfinite(ref)
        assert np.all(np.abs(got[ok] - ref[ok]) <= limit[ok])

    # results that are finite sum the same products in the order of the fp32 instruction: one rounding each
    def limit(ref_abs, maps):
        return (maps * taps + 16) * 2.0 ** -24 * np.where(np.isfinite(ref_abs), ref_abs, 0.0)

    xs, gs, ws = x.copy(), g.copy(), w.copy()
    xs[4, 5, 6, 7] = value
    gs[11, 3, 0, 8] = value
    same(p.fwd(dev(xs), dev(w)), oracle.conv3d_fwd(xs, w), limit(oracle.conv3d_fwd(np.abs(xs), np.abs(w)), f))
    same(p.bwd(dev(gs), dev(w)), oracle.conv3d_bwd(gs, w, n), limit(oracle.conv3d_bwd(np.abs(gs), np.abs(w), n), fo))
    ws[17, 3, 1, 2, 0] = value
    xw = x * 2.0 ** -10
    same(p.fwd(dev(xw), dev(ws)), oracle.conv3d_fwd(xw, ws), limit(oracle.conv3d_fwd(np.abs(xw), np.abs(ws)), f))
    p.close()


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("s", [(1, 1, 1), (2, 3, 2)])
def test_finite_results_stand_beside_those_that_are_not(value, s):
    """Maps whose weights are not finite, as in a net that has diverged, are none of the others' business; nor are single voxels."""
    f, fo, n, k = 40, 40, (21, 24, 30), (3, 3, 3)
    x, w, g = tensors(f, fo, n, k, s, 9109)
    p = znn.Plan(f, fo, n, k, "direct", s)
    assert p.workspace_bytes(0) > 0 and p.workspace_bytes(1) > 0        # packed weights
    out, gin = p.fwd(dev(x), dev(w)).cpu().numpy(), p.bwd(dev(g), dev(w)).cpu().numpy()

    def stands(got, base, ref, there, inner=slice(None)):
        got = got.cpu().numpy()
        assert np.array_equal(got[~there], base[~there])
        got, ref = got[inner], ref[inner]
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
        assert np.array_equal(np.isneginf(got), np.isneginf(ref))

    for maps in ((3, 17, 39), range(8, 40)):
        for wx, at in ((w.copy(), (list(maps),)), (w.copy(), (slice(None), list(maps)))):
            wx[at] = value
            if len(at) == 1:
                there = np.zeros(out.shape, bool)
                there[list(maps)] = True
                stands(p.fwd(dev(x), dev(wx)), out, oracle.conv3d_fwd(x, wx, s), there)
            else:
                there = np.zeros(gin.shape, bool)
                there[list(maps)] = True
                # at the border the kernels multiply weights by zeros that the oracle leaves out
                stands(p.bwd(dev(g), dev(wx)), gin, oracle.conv3d_bwd(g, wx, n, s), there,
                       (slice(None),) + tuple(slice(2 * b, a - 2 * b) for a, b in zip(n, s)))
    x[9, 7, 8, 9] = g[21, 5, 5, 5] = value
    ref = oracle.conv3d_fwd(x, w, s)
    stands(p.fwd(dev(x), dev(w)), out, ref, ~np.isfinite(ref))
    ref = oracle.conv3d_bwd(g, w, n, s)
    stands(p.bwd(dev(g), dev(w)), gin, ref, ~np.isfinite(ref))
    p.close()


GRADIENTS = [
    # f, fo, n, k, s: pieces of the axes with and without a remainder, tap groups, column groups, shares
    (1, 1, (1, 1, 5), (1, 1, 1), (1, 1, 1)),            # fewer voxels than pieces
    (1, 40, (9, 10, 11), (3, 3, 3), (1, 1, 1)),         # all taps in one group
    (3, 5, (2, 3, 50), (2, 2, 7), (1, 1, 1)),
    (16, 16, (8, 16, 32), (1, 1, 1), (1, 1, 1)),        # nothing left over anywhere
    (17, 33, (11, 13, 15), (2, 3, 4), (1, 1, 1)),
    (40, 40, (14, 13, 12), (3, 3, 3), (1, 1, 1)),
    (24, 81, (5, 20, 19), (2, 3, 4), (1, 1, 1)),        # two groups of map tiles
    (130, 7, (6, 6, 9), (2, 2, 2), (1, 1, 1)),          # column groups
    (6, 33, (1, 60, 47), (1, 11, 11), (1, 1, 1)),       # 2D
    (12, 12, (15, 14, 13), (3, 3, 3), (2, 3, 4)),       # residues of different extents
    (10, 10, (9, 9, 11), (3, 3, 3), (4, 4, 5)),         # result extents below the tap spacing
    (8, 24, (3, 30, 30), (1, 3, 3), (3, 2, 2)),         # spacing on an axis of one tap
    (5, 5, (30, 9, 10), (17, 9, 7), (1, 1, 1)),
    (4, 6, (40, 41, 42), (3, 3, 3), (1, 1, 1)),         # many shares, four sums per element
]


# As WIDE_SHAPES
WIDE_GRADIENTS = [
    (2, 40, (60, 61, 62), (3, 3, 3), (1, 1, 1)),        # all taps in one group
    (128, 128, (8, 32, 128), (1, 1, 1), (1, 1, 1)),     # nothing left over anywhere
    (17, 33, (31, 33, 35), (2, 3, 4), (1, 1, 1)),
    (24, 81, (15, 20, 29), (2, 3, 4), (1, 1, 1)),       # two groups of map tiles
    (260, 16, (26, 26, 29), (2, 2, 2), (1, 1, 1)),      # column groups
    (6, 33, (1, 160, 147), (1, 11, 11), (1, 1, 1)),     # 2D
    (40, 40, (25, 24, 23), (3, 3, 3), (2, 3, 4)),       # residues of different extents
    (64, 64, (20, 44, 45), (3, 3, 3), (9, 4, 4)),       # a result extent below the tap spacing
    (40, 48, (6, 61, 60), (1, 3, 3), (3, 2, 2)),        # spacing on an axis of one tap
    (5, 5, (40, 29, 30), (17, 9, 7), (1, 1, 1)),        # 1071 taps
    (6, 40, (40, 41, 42), (3, 3, 3), (1, 1, 1)),        # many shares
]


def gradient_within_bound(f, fo, n, k, s, *names):
    x, w, g = tensors(f, fo, n, k, s, 9103)
    p = znn.Plan(f, fo, n, k, "direct", s)
    gw = kernels_of(lambda: p.wgrad(dev(x), dev(g)), *names).cpu().numpy()
    voxels = g[0].size
    # a step per 32 voxels, remainders of pieces and tiles at most double them; waves and shares
    limit = (2 * (voxels // 32) + 600) * 2.0 ** -24 * oracle.conv3d_wgrad(np.abs(x), np.abs(g), s)
    assert np.all(np.abs(gw.astype(np.float64) - oracle.conv3d_wgrad(x, g, s)) <= limit)
    p.close()


@pytest.mark.parametrize("f,fo,n,k,s", GRADIENTS)
def test_kernel_gradient_stays_within_the_bound_of_the_split(f, fo, n, k, s):
    gradient_within_bound(f, fo, n, k, s)


@pytest.mark.parametrize("f,fo,n,k,s", WIDE_GRADIENTS)
def test_kernel_gradient_of_wide_layers_runs_on_the_split_and_stays_within_its_bound(f, fo, n, k, s):
    gradient_within_bound(f, fo, n, k, s, "split of images", "direct kernel gradient (MFMA)")


def gradient_as_in_fp32(f, fo, n, k, s, value, *names):
    x, w, g = tensors(f, fo, n, k, s, 9104)
    x[4, 5, 6, 7] = value
    g *= 2.0 ** -10
    p = znn.Plan(f, fo, n, k, "direct", s)
    got = kernels_of(lambda: p.wgrad(dev(x), dev(g)), *names).cpu().numpy().astype(np.float64)
    ref = oracle.conv3d_wgrad(x, g, s)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.array_equal(np.isneginf(got), np.isneginf(ref))
    ok = np.isfinite(ref)
    ref_abs = oracle.conv3d_wgrad(np.abs(x), np.abs(g), s)
    assert np.all(np.abs(got[ok] - ref[ok]) <= (2 * g[0].size + 600) * 2.0 ** -24 * ref_abs[ok])
    p.close()


@pytest.mark.parametrize("value", [np.inf, np.nan, 3.4e38])
@pytest.mark.parametrize("s", [(1, 1, 1), (2, 1, 2)])
def test_kernel_gradient_of_images_that_are_not_finite_acts_as_in_fp32(value, s):
    gradient_as_in_fp32(9, 20, (11, 12, 13), (3, 3, 3), s, value)


@pytest.mark.parametrize("value", [np.inf, np.nan, 3.4e38])
@pytest.mark.parametrize("n,s", [((24, 22, 27), (1, 1, 1)), ((26, 24, 29), (2, 1, 2))])
def test_kernel_gradient_of_wide_layers_that_are_not_finite_acts_as_in_fp32(value, n, s):
    gradient_as_in_fp32(40, 36, n, (3, 3, 3), s, value, "direct kernel gradient (MFMA)")


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("f,fo,n,k,s", [
    (40, 40, (26, 24, 30), (3, 3, 3), (1, 1, 1)),
    (40, 37, (28, 30, 27), (3, 3, 3), (2, 3, 2)),
    (80, 80, (1, 60, 71), (1, 11, 11), (1, 1, 1)),      # five row tiles
    (24, 81, (15, 20, 29), (2, 3, 4), (1, 1, 1)),       # two groups of them, columns that end within a tile
])
def test_finite_kernel_gradients_stand_beside_those_that_are_not(f, fo, n, k, s, value):
    x, w, g = tensors(f, fo, n, k, s, 9110)
    p = znn.Plan(f, fo, n, k, "direct", s)
    base = kernels_of(lambda: p.wgrad(dev(x), dev(g)), "direct kernel gradient (MFMA)").cpu().numpy()

    def stands(x, g, maps, limit):
        got, ref = p.wgrad(dev(x), dev(g)).cpu().numpy(), oracle.conv3d_wgrad(x, g, s)
        there = np.zeros(base.shape, bool)
        there[maps] = True
        assert np.all(np.abs(got[~there] - base[~there]) <= limit[~there])
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
        assert np.array_equal(np.isneginf(got), np.isneginf(ref))

    # whole maps of either image: no products of theirs are taken again where they are NaN.  Else those of their waves, in fp32.
    limit = (2 * g[0].size + 600) * 2.0 ** -24 * oracle.conv3d_wgrad(np.abs(x), np.abs(g), s) * 2
    whole = 0 * limit if np.isnan(value) else limit
    xs, gs = x.copy(), g.copy()
    xs[5] = gs[17] = value
    stands(xs, g, np.s_[:, 5], whole)
    stands(x, gs, np.s_[17], whole)
    xs, gs = x.copy(), g.copy()
    xs[3, :, -3, 9] = gs[2, 0, 0, -1] = value           # some voxels
    stands(xs, g, np.s_[:, 3], limit)
    stands(x, gs, np.s_[2], limit)
    p.close()


@pytest.mark.parametrize("f,fo,n,k,s", [
    (8, 8, (131, 120, 121), (3, 3, 3), (1, 1, 1)),      # slabs of planes
    (16, 16, (1, 1100, 1001), (1, 3, 3), (1, 1, 1)),    # slabs of rows
    (16, 16, (80, 121, 120), (3, 2, 2), (3, 2, 2)),     # slabs of one residue
    (8, 9, (1, 1300, 1201), (1, 3, 2), (1, 1, 1)),      # on the vector ALUs
    (6, 8, (140, 121, 120), (3, 2, 2), (3, 2, 2)),
])
def test_kernel_gradient_of_large_layers_in_slabs(f, fo, n, k, s):
    x, w, g = tensors(f, fo, n, k, s, 9105)
    p = znn.Plan(f, fo, n, k, "direct", s)
    assert (f * x[0].size + fo * g[0].size) * 6 * 1.2 > 96 << 20 and p.workspace_bytes(2) < 192 << 20
    gw = kernels_of(lambda: p.wgrad(dev(x), dev(g)), "direct kernel gradient (%s)" % ("few maps" if f * fo < 64 or fo == 9 else "MFMA")).cpu().numpy()
    ref, ref_abs = oracle.conv3d_wgrad(x, g, s), oracle.conv3d_wgrad(np.abs(x), np.abs(g), s)
    # sums this long are far inside the worst case: a tenth of it still leaves a lost or doubled slab no room
    assert np.all(np.abs(gw.astype(np.float64) - ref) <= 0.1 * (2 * (g[0].size // 32) + 600) * 2.0 ** -24 * ref_abs)
    p.close()


@pytest.mark.parametrize("f,fo,n,k,s", [
    (16, 16, (1, 1, 1200000), (1, 1, 5), (1, 1, 1)),    # pieces of 150 000 vectors
    (16, 16, (1, 1, 1300001), (1, 1, 5), (1, 1, 2)),    # two residues of pieces of 81 000
])
def test_kernel_gradient_of_long_rows(f, fo, n, k, s):
    x, w, g = tensors(f, fo, n, k, s, 9107)
    p = znn.Plan(f, fo, n, k, "direct", s)
    assert p.workspace_bytes(2) > 4 * (x.size + g.size)                 # copies of the images
    gw = p.wgrad(dev(x), dev(g)).cpu().numpy()
    ref, ref_abs = oracle.conv3d_wgrad(x, g, s), oracle.conv3d_wgrad(np.abs(x), np.abs(g), s)
    # The sums walk randomly, some 1e-3 of ref_abs far, and so do their roundings: 2^-24 1e-3 sqrt(voxels / 32) is 1e-8 of it.  32 wrong
    # voxels of a million (four vectors) are off by sqrt(32) / 3 products of size 1, 6e-6 of it.
    assert np.all(np.abs(gw.astype(np.float64) - ref) <= 5e-7 * ref_abs)
    p.close()
