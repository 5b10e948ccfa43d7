"""The forward entry point that allocates nothing (built-in scratch array) against the ordinary
one with a caller workspace: same kernels, so outputs must agree bit for bit; and against the
oracle, to the tolerance of the method."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1510_06706_amd import binding as znn
from paper_1510_06706_amd import synth

pytestmark = pytest.mark.gpu

TOL = {"direct": 1e-4, "fft": 1e-3}

# two calls in a row on the same GPU, the second with a smaller input; the first direct-method
# shape splits its input maps over workgroups, so partial sums go through the scratch as well
CALLS = [(12, 24, (20, 21, 22), (3, 3, 3)), (5, 7, (12, 13, 14), (2, 3, 2))]


@pytest.mark.parametrize("mode", ["direct", "fft"])
def test_forward_without_allocation_matches_forward_with_workspace(mode):
    import torch
    dev = torch.device("cuda:0")
    for call, (f, fo, n, k) in enumerate(CALLS):
        cfg = synth.LayerShape("noalloc", f, fo, n, k, 1.0 / np.sqrt(f * np.prod(k)), 700 + call)
        inp, w, _ = synth.layer_tensors(cfg)
        d_in, d_w = torch.from_numpy(inp).to(dev), torch.from_numpy(w).to(dev)
        p = znn.Plan(f, fo, n, k, mode)
        assert 0 < p.workspace_bytes(znn.ZNN_PASS_FWD) <= znn.STATIC_SCRATCH_BYTES
        want = p.fwd(d_in, d_w)
        got = torch.full_like(want, float("nan"))
        torch.cuda.synchronize()
        # torch's allocator counts every block it hands out: the call must not add to that count
        # (bytes in use may drop meanwhile, when the collector frees tensors of earlier tests)
        before = torch.cuda.memory_stats(dev)["allocation.all.allocated"]
        p.fwd_static(d_in, d_w, got)
        torch.cuda.synchronize()
        assert torch.cuda.memory_stats(dev)["allocation.all.allocated"] == before
        assert torch.equal(got, want), (mode, call)
        ref = oracle.conv3d_fwd(inp, w)
        err = float(np.max(np.abs(got.cpu().numpy().astype(np.float64) - ref)) / np.max(np.abs(ref)))
        print("no-alloc forward %s call %d: rel-err %.2e" % (mode, call, err), flush=True)
        assert err <= TOL[mode]
        p.close()


# layers whose tiles take more than the array where whole volumes would not: kernels transformed by the call, and resident
TILES = [(1, 15, (77, 47, 81), (3, 3, 3), False), (15, 42, (69, 22, 58), (1, 5, 5), False), (10, 1, (80, 80, 80), (3, 3, 3), False),
         (75, 4, (39, 39, 39), (6, 6, 6), True), (105, 9, (1, 286, 240), (1, 3, 3), True), (24, 25, (54, 54, 54), (5, 5, 5), True)]


@pytest.mark.parametrize("f,fo,n,k,resident", TILES)
def test_forward_without_allocation_takes_the_tiles_of_a_layer_in_groups(f, fo, n, k, resident):
    import torch
    print("case", f, fo, n, k, resident, flush=True)
    dev = torch.device("cuda:0")
    inp, w, gout = synth.layer_tensors(synth.LayerShape("noalloc", f, fo, n, k, 1.0 / np.sqrt(f * np.prod(k)), 710 + f))
    d_in, d_w, d_g = (torch.from_numpy(a).to(dev) for a in (inp, w, gout))
    p = znn.Plan(f, fo, n, k, "fft")
    assert p.tiles is not None
    if resident:
        p.prepare_kernels(d_w)
    w_ = None if resident else d_w
    assert p.workspace_bytes(znn.ZNN_PASS_FWD) > znn.STATIC_SCRATCH_BYTES
    want = p.fwd(d_in, w_)
    got = torch.full_like(want, float("nan"))
    p.fwd_static(d_in, w_, got)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    # node spectra for a memoized kernel gradient are left whole
    gw = p.wgrad(d_in, d_g)
    p.enable_memo()
    p.bwd(d_g, w_)
    p.fwd_static(d_in, w_, got.fill_(float("nan")))
    assert torch.equal(got, want) and torch.equal(p.wgrad_memo(), gw)
    p.close()


def test_forward_without_allocation_refuses_layers_beyond_the_array():
    import torch
    cfg = synth.CONFIG2
    p = znn.Plan(cfg.fan_in, cfg.fan_out, cfg.image, cfg.kernel, "fft")
    assert p.workspace_bytes(znn.ZNN_PASS_FWD) > znn.STATIC_SCRATCH_BYTES
    x = torch.zeros((cfg.fan_in,) + cfg.image, dtype=torch.float32, device="cuda:0")
    w = torch.zeros((cfg.fan_out, cfg.fan_in) + cfg.kernel, dtype=torch.float32, device="cuda:0")
    out = torch.zeros((cfg.fan_out,) + cfg.out, dtype=torch.float32, device="cuda:0")
    rc = znn.lib().znn_conv3d_fwd_static(p._h, ctypes.c_void_p(x.data_ptr()), ctypes.c_void_p(w.data_ptr()),
                                         ctypes.c_void_p(out.data_ptr()), ctypes.c_void_p(0))
    assert rc == znn.ZNN_EWORKSPACE and "built-in array" in znn.last_error()
    p.close()


# layers of the direct method whose weights, or sums of the shares of their input maps, take more than the array: three groups of maps
# (the last one smaller), shares of the input maps as well, and a layer whose weights of sixteen output maps do not fit; shares of the
# input maps a few at a time, one at a time, and none, as the sums of one do not fit
WIDE = [(200, 213, (6, 9, 20), (5, 5, 5), True), (160, 120, (8, 9, 12), (7, 7, 7), True), (512, 3, (9, 9, 10), (9, 9, 9), False),
        (400, 16, (36, 36, 36), (9, 9, 9), True), (440, 16, (36, 36, 36), (9, 9, 9), True), (470, 16, (36, 36, 36), (9, 9, 9), False)]


@pytest.mark.parametrize("f,fo,n,k,same", WIDE)
def test_forward_without_allocation_takes_the_output_maps_of_a_layer_in_groups(f, fo, n, k, same):
    import torch
    print("case", f, fo, n, k, flush=True)
    x = torch.rand((f,) + n, device="cuda:0") * 2 - 1
    w = torch.rand((fo, f) + k, device="cuda:0") * 2 - 1
    p = znn.Plan(f, fo, n, k, "direct")
    assert not same or p.workspace_bytes(znn.ZNN_PASS_FWD) > znn.STATIC_SCRATCH_BYTES
    want = p.fwd(x, w)
    got = torch.full_like(want, float("nan"))
    p.fwd_static(x, w, got)
    torch.cuda.synchronize()
    assert torch.equal(got, want) or not same
    # sums of f k^3 rounded products in two orders
    size = p.fwd(x.abs(), w.abs())
    assert bool(((got - want).abs() <= 2.0 ** -23 * (f * k[0] * k[1] * k[2]) ** 0.5 * 4 * size).all())
    p.close()
