"""The direct kernels on the vector ALUs (one or two input-side maps, small layers, shapes the matrix kernels do not take):
widths of their tap groups, blocks of maps, shares of the voxels.

Bounds are derived from S = sum of |products|: one rounding per product and sum, in chains of fp32 multiply-adds.
"""
import numpy as np
import pytest

import oracle
from paper_1510_06706_amd import binding as znn
from paper_1510_06706_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = [
    # f, fo, n, k, s: groups of 1, 2, 3, 4, 5, 7 and 11 taps along x, maps around the blocks of 4 and 8
    (1, 1, (4, 5, 6), (1, 1, 1), (1, 1, 1)),
    (1, 4, (16, 16, 16), (3, 3, 3), (1, 1, 1)),
    (1, 5, (6, 7, 40), (2, 1, 13), (1, 1, 1)),
    (2, 9, (5, 9, 30), (1, 3, 22), (1, 1, 1)),
    (1, 17, (3, 12, 31), (2, 4, 10), (1, 1, 1)),
    (1, 8, (9, 8, 33), (3, 2, 8), (1, 1, 1)),
    (7, 1, (9, 8, 33), (1, 2, 7), (1, 1, 1)),           # backward: one map on the input side
    (1, 3, (21, 23, 25), (3, 2, 3), (2, 5, 4)),         # sparse taps
    (1, 6, (1, 90, 91), (1, 11, 11), (1, 1, 1)),        # 2D, several shares
    (2, 2, (40, 41, 43), (3, 3, 3), (1, 1, 1)),         # several shares
    (1, 1, (18, 18, 17), (17, 17, 15), (1, 1, 1)),      # 4335 taps
]


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a.astype(np.float32))).to("cuda:0")


@pytest.mark.parametrize("f,fo,n,k,s", SHAPES)
def test_passes_stay_within_the_bound_of_fp32_chains(f, fo, n, k, s):
    x, w, g = synth.layer_tensors(synth.LayerShape("t", f, fo, n, k, 1.0, 9200, s))
    taps, eps = k[0] * k[1] * k[2], 2.0 ** -24
    p = znn.Plan(f, fo, n, k, "direct", s)

    def close(got, ref, ref_abs, terms):
        assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= (terms + 16) * eps * ref_abs)

    a, b, c = np.abs(x), np.abs(w), np.abs(g)
    close(p.fwd(dev(x), dev(w)), oracle.conv3d_fwd(x, w, s), oracle.conv3d_fwd(a, b, s), f * taps)
    close(p.bwd(dev(g), dev(w)), oracle.conv3d_bwd(g, w, n, s), oracle.conv3d_bwd(c, b, n, s), fo * taps)
    # chains of a thread, then its workgroup's tree and the shares
    close(p.wgrad(dev(x), dev(g)), oracle.conv3d_wgrad(x, g, s), oracle.conv3d_wgrad(a, c, s), g[0].size // 64 + 32)
    p.close()


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("n", [(9, 10, 11), (62, 63, 51)])          # one voxel a thread, four
def test_values_that_are_not_finite_reach_the_results_they_belong_to(n, value):
    f, fo, k = 1, 4, (3, 3, 3)
    x, w, g = synth.layer_tensors(synth.LayerShape("t", f, fo, n, k, 1.0, 9201))
    x[0, 4, 5, 6] = x[0, 1, 2, -3] = value
    g[2, 3, 3, 3] = g[1, 0, 1, -2] = value
    p = znn.Plan(f, fo, n, k, "direct")
    got = (p.fwd(dev(x), dev(w)), p.bwd(dev(g), dev(w)), p.wgrad(dev(x), dev(np.ones_like(g))))
    ref = (oracle.conv3d_fwd(x, w), oracle.conv3d_bwd(g, w, n), oracle.conv3d_wgrad(x, np.ones_like(g)))
    for a, b in zip(got, ref):
        a = a.cpu().numpy()
        assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isposinf(a), np.isposinf(b))
        assert np.array_equal(np.isneginf(a), np.isneginf(b))
    p.close()


@pytest.mark.parametrize("f,fo,n,k,s", [
    (1, 41, (42, 60, 12), (3, 3, 3), (1, 1, 1)),            # rows of 10: the last group repeats two voxels
    (1, 40, (66, 130, 6), (3, 3, 3), (1, 1, 1)),            # of 4, one group
    (2, 33, (66, 70, 9), (1, 2, 5), (1, 3, 1)),             # of 5, one voxel beyond it
    (1, 39, (50, 50, 17), (2, 2, 2), (3, 2, 10)),           # of 7, taps ten apart
    (1, 3, (101, 203, 8), (2, 1, 1), (1, 1, 1)),            # blocks of four maps
    (1, 40, (1, 310, 215), (1, 1, 11), (1, 1, 1)),
    (3, 4, (90, 90, 20), (1, 1, 14), (1, 1, 1)),            # two groups of seven taps
    (1, 40, (90, 130, 5), (1, 1, 3), (1, 1, 1)),            # rows of 3 go voxel by voxel
])
def test_forward_passes_of_four_voxels_a_thread(f, fo, n, k, s):
    """Large passes, and a transfer function inside them."""
    import torch
    from paper_1510_06706_amd import program as zp
    print("case", f, fo, n, k, s, flush=True)
    x, w, _ = synth.layer_tensors(synth.LayerShape("t", f, fo, n, k, 1.0, 9700 + f, s))
    p = znn.Plan(f, fo, n, k, "direct", s)
    got = p.fwd(dev(x), dev(w))
    ref, size = oracle.conv3d_fwd(x, w, s), oracle.conv3d_fwd(np.abs(x), np.abs(w), s)
    assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= 2.0 ** -24 * (f * np.prod(k) + 1) * size)
    bias, out, y = torch.linspace(-0.3, 0.3, fo, device="cuda:0"), torch.empty_like(got), torch.empty_like(got)
    P = zp.Program("cuda:0", 1)
    t = [dev(x), dev(w), out, bias, y]
    for v in t:
        P.buffer("given", v.shape)
    P.add(zp.CONV_FWD, (0, 1, 2, 3, 4), plan=p)
    P.build().run(dict(enumerate(t)))
    assert torch.equal(out, got) and torch.equal(y, torch.relu(got + bias.view(-1, 1, 1, 1)))
    p.close()


@pytest.mark.parametrize("f,fo,n,k,s", [
    (41, 1, (42, 60, 10), (3, 3, 3), (1, 1, 1)),            # rows of 10: the last group repeats two voxels
    (40, 1, (66, 130, 4), (3, 3, 3), (1, 1, 1)),            # of 4, one group
    (33, 2, (66, 70, 5), (1, 2, 5), (1, 3, 1)),             # of 5, kernels as wide
    (39, 1, (50, 50, 17), (2, 2, 1), (3, 2, 1)),            # one tap a row
    (3, 1, (101, 203, 8), (2, 1, 4), (1, 1, 1)),            # blocks of four maps
    (40, 1, (1, 310, 215), (1, 1, 11), (1, 1, 1)),
    (4, 3, (90, 90, 20), (1, 1, 14), (1, 1, 1)),            # two groups of seven taps
    (40, 1, (50, 50, 17), (2, 2, 2), (1, 1, 3)),            # spaced taps go voxel by voxel
])
@pytest.mark.parametrize("in_place", [False, True])
def test_backward_passes_of_four_voxels_a_thread(f, fo, n, k, s, in_place):
    """Large passes, alone and times the derivative of a rectifier whose result they may replace."""
    import torch
    from paper_1510_06706_amd import program as zp
    print("case", f, fo, n, k, s, in_place, flush=True)
    x, w, g = synth.layer_tensors(synth.LayerShape("t", f, fo, n, k, 1.0, 9800 + f, s))
    p = znn.Plan(f, fo, n, k, "direct", s)
    got = p.bwd(dev(g), dev(w))
    ref, size = oracle.conv3d_bwd(g, w, n, s), oracle.conv3d_bwd(np.abs(g), np.abs(w), n, s)
    assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - ref) <= 2.0 ** -24 * (fo * np.prod(k) + 1) * size)
    below = torch.relu(dev(x))
    want = torch.where(below > 0, got, torch.zeros_like(got))
    P = zp.Program("cuda:0", 1)
    t = [dev(g), dev(w), below if in_place else torch.empty_like(got), below]
    for v in t:
        P.buffer("given", v.shape)
    P.add(zp.CONV_BWD, (0, 1, 2, 3), plan=p)
    P.build().run(dict(enumerate(t)))
    assert torch.equal(t[2], want)
    p.close()
