"""Products of the FFT method on overlapping tiles: workgroups of one to three result tiles of 16, sums of a length around their chunks
of four and eight.

The bound, on 2-norms: three transforms of T points round at most 6 log2 T times in a row, a product sums K terms one after another,
each rounding 2^-24 of what is at most the result of the operands' absolute values.
"""
import numpy as np
import pytest

import oracle
from paper_1510_06706_amd import binding as znn
from paper_1510_06706_amd import synth

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a.astype(np.float32))).to("cuda:0")


@pytest.mark.parametrize("f,fo,n,k", [
    (7, 15, (1, 33, 30), (1, 7, 7)),        # sums of 7, 15 and 8 tiles, results below one tile of 16
    (8, 16, (1, 40, 33), (1, 7, 5)),        # exactly one chunk, one tile
    (9, 17, (1, 52, 47), (1, 11, 11)),      # one more of each
    (23, 33, (1, 60, 44), (1, 9, 9)),
    (16, 31, (10, 18, 20), (3, 3, 3)),
    (25, 8, (12, 14, 31), (5, 4, 3)),
    (1, 16, (1, 99, 99), (1, 11, 11)),      # sums of one term
    (15, 48, (1, 99, 99), (1, 11, 11)),
])
def test_products_of_few_tiles_match_the_oracle(f, fo, n, k):
    print("case", f, fo, n, k, flush=True)
    x, w, g = synth.layer_tensors(synth.LayerShape("t", f, fo, n, k, 1.0, 9300 + f, (1, 1, 1)))
    p = znn.Plan(f, fo, n, k, "fft")
    m, t = p.tiles
    a = [np.abs(v) for v in (x, w, g)]
    for got, ref, size, terms in (
            (p.fwd(dev(x), dev(w)), oracle.conv3d_fwd(x, w), oracle.conv3d_fwd(a[0], a[1]), f),
            (p.bwd(dev(g), dev(w)), oracle.conv3d_bwd(g, w, n), oracle.conv3d_bwd(a[2], a[1], n), fo),
            (p.wgrad(dev(x), dev(g)), oracle.conv3d_wgrad(x, g), oracle.conv3d_wgrad(a[0], a[2]), int(np.prod(t)))):
        err = np.linalg.norm(got.cpu().numpy().astype(np.float64) - ref)
        assert err <= 2.0 ** -24 * (6 * np.log2(np.prod(m)) + terms) * np.linalg.norm(size)
    p.close()


# sums of one to nine chunks of four, whole and not, on 16 x 16 results and, of wide layers, on 32 x 32
@pytest.mark.parametrize("f,fo,n,k", [
    (2, 3, (1, 50, 50), (1, 5, 5)),
    (4, 5, (9, 30, 21), (3, 3, 3)),
    (11, 12, (1, 60, 33), (1, 7, 7)),
    (13, 21, (12, 14, 31), (3, 4, 3)),
    (33, 66, (58, 58, 44), (3, 3, 3)),
    (35, 97, (58, 44, 47), (4, 3, 5)),
    (61, 63, (70, 70, 70), (5, 5, 5)),          # forward and backward by 32 x 32
    (63, 127, (42, 42, 42), (7, 7, 7)),
])
def test_products_of_every_number_of_chunks_match_the_direct_method(f, fo, n, k):
    print("case", f, fo, n, k, flush=True)
    x, w, g = (dev(v) for v in synth.layer_tensors(synth.LayerShape("t", f, fo, n, k, 1.0, 9400 + f, (1, 1, 1))))
    p, q = znn.Plan(f, fo, n, k, "fft"), znn.Plan(f, fo, n, k, "direct")
    m, t = p.tiles
    for name, a, b, terms in (("fwd", x, w, f), ("bwd", g, w, fo), ("wgrad", x, g, int(np.prod(t)))):
        got, ref = getattr(p, name)(a, b).double(), getattr(q, name)(a, b).double()
        size = getattr(q, name)(a.abs(), b.abs()).double().norm()
        # the direct method sums a few thousand products, or n^3 of a gradient in shares, each chain no longer than 512
        assert (got - ref).norm() <= 2.0 ** -24 * (6 * np.log2(np.prod(m)) + terms + 512) * size, name
    p.close()
    q.close()


@pytest.mark.parametrize("f,fo,n,k,s", [
    (7, 5, (9, 31, 33), (3, 4, 3), (1, 1, 1)),          # few entries: none are doubled up
    (34, 40, (1, 90, 77), (1, 7, 9), (1, 1, 1)),        # 2D, clipped tiles, kernels by twice the waves and entries
    (48, 40, (23, 40, 42), (3, 5, 5), (1, 1, 1)),
    (24, 25, (26, 30, 44), (2, 3, 2), (2, 3, 4)),       # spaced taps
    (40, 30, (30, 33, 62), (11, 9, 12), (1, 1, 1)),     # tiles of 32
])
def test_transforms_of_both_operands_in_one_launch(f, fo, n, k, s):
    """Kernels transformed beside the images, and images beside the gradients, give the bits of launches of their own
    (prepared kernels, kept node spectra)."""
    import torch
    print("case", f, fo, n, k, s, flush=True)
    x, w, g = (dev(v) for v in synth.layer_tensors(synth.LayerShape("t", f, fo, n, k, 1.0, 9500 + f, s)))
    p, q = znn.Plan(f, fo, n, k, "fft", s), znn.Plan(f, fo, n, k, "fft", s)
    assert p.tiles is not None
    q.enable_memo("cuda:0")
    q.prepare_kernels(w)
    assert torch.equal(p.fwd(x, w), q.fwd(x, None))
    assert torch.equal(p.bwd(g, w), q.bwd(g, None))
    assert torch.equal(p.wgrad(x, g), q.wgrad_memo())
    p.close()
    q.close()


# images of one tile (the inverse transform itself takes the derivative) and of many, windows that let samples travel by four, two and one
@pytest.mark.parametrize("f,fo,n,k", [(5, 7, (1, 20, 22), (1, 5, 5)), (17, 6, (9, 40, 37), (2, 4, 4)), (8, 9, (1, 66, 71), (1, 6, 7)),
                                      (33, 34, (11, 33, 60), (3, 5, 5)), (4, 3, (1, 40, 40), (1, 13, 13)), (8, 9, (8, 12, 12), (1, 9, 9))])
def test_transfer_functions_inside_the_passes_give_the_bits_of_their_own(f, fo, n, k):
    import torch
    from paper_1510_06706_amd import program as zp
    print("case", f, fo, n, k, flush=True)
    x, w, g = (dev(v) for v in synth.layer_tensors(synth.LayerShape("t", f, fo, n, k, 1.0, 9600 + f, (1, 1, 1))))
    p = znn.Plan(f, fo, n, k, "fft")
    assert p.tiles is not None
    bias = torch.linspace(-0.2, 0.3, fo, device="cuda:0")
    below = torch.where(x > 0, x, torch.zeros_like(x))           # a rectifier's result
    out, gin, y = torch.empty_like(g), torch.empty_like(x), torch.empty_like(g)
    P = zp.Program("cuda:0", 1)
    for t in (x, w, out, bias, y, g, gin, below):
        P.buffer("given", t.shape)
    P.add(zp.CONV_FWD, (0, 1, 2, 3, 4), plan=p)
    P.add(zp.CONV_BWD, (5, 1, 6, 7), plan=p)
    P.build().run(dict(enumerate([x, w, out, bias, y, g, gin, below])))
    ref, back = p.fwd(x, w), p.bwd(g, w)
    assert torch.equal(out, ref) and torch.equal(y, torch.relu(ref + bias.view(-1, 1, 1, 1)))
    assert torch.equal(gin, torch.where(below > 0, back, torch.zeros_like(back)))
    p.close()


# inverse transforms with columns of 32 by workgroups of two and of four waves, of one tile and of seven
@pytest.mark.parametrize("f,fo,n,k", [(1, 87, (41, 41, 29), (2, 3, 2)), (3, 87, (32, 23, 17), (4, 4, 4)), (6, 79, (1, 194, 179), (1, 11, 11)),
                                      (1, 36, (47, 17, 31), (4, 4, 4)), (1, 82, (1, 172, 136), (1, 11, 11))])
def test_inverse_transforms_of_long_columns_match_the_direct_method(f, fo, n, k):
    print("case", f, fo, n, k, flush=True)
    for f, fo in ((f, fo), (fo, f)):
        x, w, g = (dev(v) for v in synth.layer_tensors(synth.LayerShape("t", f, fo, n, k, 1.0, 9900 + f, (1, 1, 1))))
        p, q = znn.Plan(f, fo, n, k, "fft"), znn.Plan(f, fo, n, k, "direct")
        assert 32 in p.tiles[0]
        for name, a, b, terms in (("fwd", x, w, f), ("bwd", g, w, fo)):
            got, ref = getattr(p, name)(a, b).double(), getattr(q, name)(a, b).double()
            size = getattr(q, name)(a.abs(), b.abs()).double().norm()
            # the direct method sums at most a few thousand products in chains no longer than 512
            assert (got - ref).norm() <= 2.0 ** -24 * (6 * np.log2(np.prod(p.tiles[0])) + terms + 512) * size, name
        p.close()
        q.close()
