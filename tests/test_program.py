"""Programs (znn_program_*): a list of operations run as one call gives what the same list gives operation by operation.

The lists here are ones that no net emits: every order that the operations allow, and buffers used again."""
import itertools

import numpy as np
import pytest

from paper_1510_06706_amd import binding as znn
from paper_1510_06706_amd import program as zp

SHAPE = (3, 10, 12, 9)          # of every image; kernels of one voxel keep it


def program(ops, shapes):
    """ops: (kind, buffers, options of Program.add); all buffers are given to the run."""
    P = zp.Program("cuda:0")
    for s in shapes:
        P.buffer("given", s)
    for kind, buf, how in ops:
        P.add(kind, buf, **how)
    return P.build()


def conv_shapes(plan):
    """in, w, out, gout, gin, gw"""
    i, o, w = (plan.f,) + plan.n, (plan.fo,) + plan.o, (plan.fo, plan.f) + plan.k
    return [i, w, o, o, i, w]


def conv_ops(plan, order):
    ops = {"F": (zp.CONV_FWD, (0, 1, 2), dict(plan=plan)), "B": (zp.CONV_BWD, (3, 1, 4), dict(plan=plan)),
           "W": (zp.CONV_WGRAD, (0, 3, 5), dict(plan=plan))}
    return [ops[c] for c in order]


ORDERS = ["".join(o) for o in itertools.permutations("FBW")]


def test_spectra_are_shared_only_by_passes_that_follow_the_ones_that_make_them():
    plan = znn.Plan(8, 8, (24, 24, 24), (3, 3, 3), "fft")
    need = lambda ops, more=(): program(ops, conv_shapes(plan) + list(more)).scratch_bytes  # noqa: E731
    memo, spectra = plan.memo_bytes(), plan.spectra_bytes()
    both = need(conv_ops(plan, "FBW"))
    assert both == memo + spectra + plan.workspace_bytes(znn.ZNN_PASS_WGRAD)
    for o in ORDERS:
        assert need(conv_ops(plan, o)) == both - (memo if o[-1] != "W" else 0), o
    # nor are they once something has written the values they were made of
    F, B, W = conv_ops(plan, "FBW")
    alone = max(plan.workspace_bytes(w) for w in (znn.ZNN_PASS_FWD, znn.ZNN_PASS_BWD, znn.ZNN_PASS_WGRAD))
    for buffer, ops, want in ((0, lambda t: [F, t, B, W], both - memo), (3, lambda t: [F, B, t, W], both - memo),
                              (1, lambda t: [F, t, B, W], memo + alone), (1, lambda t: [t, F, B, W], both),
                              (0, lambda t: [t, B, F, W], both), (3, lambda t: [F, t, B, W], both)):
        shape = conv_shapes(plan)[buffer]
        write = (zp.TRANSFER_FWD, (6, 7, buffer), dict(maps=shape[0], n=(1, 1, int(np.prod(shape[1:])))))
        assert need(ops(write), [shape, shape[:1]]) == want, buffer


# ------------------------------------------------------------------------------------------------------- on the GPU
def step_by_step(ops, t):
    """The list through the single entry points, on tensors t."""
    names = {v: k for k, v in znn.TRANSFER_FNS.items()}
    assert len(names) == len(znn.TRANSFER_FNS)
    for kind, b, how in ops:
        b, fn = list(b) + [-1] * (8 - len(b)), how.get("fn", "rectify")
        if kind == zp.CONV_FWD:
            how["plan"].fwd(t[b[0]], t[b[1]], t[b[2]])
            if b[4] >= 0:
                t[b[4]].copy_(znn.transfer_fwd(t[b[2]], t[b[3]], fn))
        elif kind == zp.CONV_BWD:
            how["plan"].bwd(t[b[0]], t[b[1]], t[b[2]])
            if b[3] >= 0:
                t[b[2]].copy_(znn.transfer_bwd(t[b[2]], t[b[3]], fn))
        elif kind == zp.CONV_WGRAD:
            how["plan"].wgrad(t[b[0]], t[b[1]], t[b[2]])
        elif kind == zp.TRANSFER_FWD:
            t[b[2]].copy_(znn.transfer_fwd(t[b[0]], t[b[1]], fn))
        elif kind == zp.TRANSFER_BWD:
            t[b[2]].copy_(znn.transfer_bwd(t[b[0]], t[b[1]], fn))
        elif kind == zp.BIAS_GRAD:
            t[b[1]].copy_(znn.bias_grad(t[b[0]]))
        elif kind == zp.NODE_SUM:
            total = t[b[1]].clone()
            for q in b[2:7]:
                if q >= 0:
                    znn.accumulate(total, t[q])
            t[b[0]].copy_(total if b[7] < 0 else znn.transfer_bwd(total, t[b[7]], fn))
        else:
            assert kind == zp.UPDATE
            znn.sgd_update(t[b[1]], t[b[0]], ETA)


ETA = 0.125


def check(ops, shapes, seed, runs=2, same=()):
    """Every buffer after every run, with new values before each; `same`: pairs of buffers that are one tensor."""
    import torch
    P = program(ops, shapes)
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    for r in range(runs):
        got = [torch.rand(s, generator=gen, device="cuda:0") * 2 - 1 for s in shapes]
        ref = [t.clone() for t in got]
        for a, b in same:
            got[b], ref[b] = got[a], ref[a]
        P.run(dict(enumerate(got)), ETA)
        step_by_step(ops, ref)
        torch.cuda.synchronize()
        for b, (x, y) in enumerate(zip(got, ref)):
            x, y = x.cpu().numpy().astype(np.float64), y.cpu().numpy().astype(np.float64)
            # 32-bit sums of up to 1080 terms in another order
            assert np.max(np.abs(x - y)) <= 2e-5 * max(np.max(np.abs(y)), 1e-3), (r, b)


@pytest.mark.gpu
@pytest.mark.parametrize("layout", ["auto", "full"])
@pytest.mark.parametrize("order", ORDERS)
def test_passes_of_a_layer_in_every_order(order, layout):
    print("case", order, layout, flush=True)
    plan = znn.Plan(4, 5, (14, 12, 15), (3, 2, 3), "fft")
    plan.set_spectra_layout(layout)
    assert (plan.tiles is None) == (layout != "auto")
    check(conv_ops(plan, order), conv_shapes(plan), 1)


@pytest.mark.gpu
@pytest.mark.parametrize("buffer", [0, 1, 3])
@pytest.mark.parametrize("order", ["FBW", "BFW"])
def test_operands_of_a_layer_written_between_its_passes(order, buffer):
    print("case", order, buffer, flush=True)
    plan = znn.Plan(4, 5, (14, 12, 15), (3, 2, 3), "fft")
    shapes = conv_shapes(plan)
    shape = shapes[buffer]
    maps, n = shape[0], (1, 1, int(np.prod(shape[1:]))) if len(shape) > 4 else shape[1:]
    write = (zp.TRANSFER_FWD, (6, 7, buffer), dict(maps=maps, n=n, fn="tanh"))
    ops = conv_ops(plan, order)
    for at in (1, 2):
        check(ops[:at] + [write] + ops[at:], shapes + [shape, (maps,)], 2 + at)
