"""Performance cases of the convolutional-layer library: what its users have it do, over the sizes they use.

A case is a dict of plain values.  Four kinds of work go through the public entry points:

  layer   one fully connected convolutional layer trained once through ``binding.Plan``: forward, backward
          and kernel gradient by the direct or by the FFT method.  ``memo`` (FFT only) is the memoized
          schedule: kernels transformed once, node spectra of the two passes kept for the gradient.
  train   one training round of a layered net through ``net.Net`` (forward, loss gradient, backward,
          update), launched eagerly or (``replay``) recorded once into a HIP graph and replayed.
  infer   the forward pass of a layered net alone: dense prediction on a block of a volume.
  graph   one training round of a branching multi-scale net through ``graph.GraphNet``.

Layers are described by map counts f -> fo, image extents nz ny nx, kernel extents kz ky kx and the tap
spacing s; nets by their family, their width and the extent of their output patch.
"""
import math

import torch

from paper_1510_06706_amd import binding as znn
from paper_1510_06706_amd import graph as zgraph
from paper_1510_06706_amd import net as znet
from paper_1510_06706_amd import synth

DEV = "cuda:0"


# ------------------------------------------------------------------------------------------ descriptions
def _layer(f, fo, n, k, method, memo=False, s=1, **more):
    return dict(kind="layer", f=f, fo=fo, nz=n[0], ny=n[1], nx=n[2], kz=k[0], ky=k[1], kx=k[2], s=s,
                method=method, memo=memo, **more)


def listed():
    return [
        # The smallest layer in use: a first layer on one small patch.  Three calls, a few microseconds each.
        _layer(1, 4, (16, 16, 16), (3, 3, 3), "direct", name="layer_first_direct"),
        # A wide 3D layer of the middle of a net, in both methods.
        _layer(40, 40, (64, 64, 64), (5, 5, 5), "direct", name="layer_wide_direct"),
        _layer(40, 40, (64, 64, 64), (5, 5, 5), "fft", True, name="layer_wide_fft"),
        # A wide 2D layer with large kernels, where the FFT method is the one to use.
        _layer(80, 80, (1, 256, 256), (1, 11, 11), "fft", True, name="layer_2d_fft"),
        # The widest layer a single GPU is used for, by the method the autotuner picks for it.
        _layer(120, 120, (96, 96, 96), (7, 7, 7), "fft", True, name="layer_widest_fft"),
        # Anisotropic volumes (thick sections: fewer, coarser voxels along z) cut at no round size, in both
        # methods; the FFT one as a net without memoization runs it, transforms inside every pass.
        _layer(24, 36, (23, 75, 61), (3, 5, 5), "direct", name="layer_ragged_direct"),
        _layer(20, 28, (23, 131, 115), (3, 7, 7), "fft", name="layer_ragged_fft"),
        # One round of the six-layer 3D net on the usual 12^3 output patch, launched eagerly.
        dict(kind="train", family="3d", width=40, patch=12, replay=False, name="train_3d"),
        # The 2D net with 11 x 11 kernels and a 48 x 48 output patch, launched eagerly.
        dict(kind="train", family="2d", width=40, patch=48, replay=False, name="train_2d"),
        # The max-filtering net (sparse convolutions) that stands for a sliding-window pooling net: the same
        # round recorded into a HIP graph, as long training runs do.
        dict(kind="train", family="3d_sparse", width=40, patch=12, replay=True, name="train_3d_sparse_replay"),
        # Dense prediction with that net on one block of a volume.
        dict(kind="infer", family="3d_sparse", width=40, patch=33, name="infer_3d_sparse"),
        # Three branches of different sparsity converging on a node, two outputs, several streams.
        dict(kind="graph", width=40, n=40, name="graph_multiscale"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_layer(rng):
    f = 1 if rng.random() < 0.12 else _log_int(rng, 4, 120)
    fo = rng.randint(1, 4) if rng.random() < 0.12 else _log_int(rng, 4, 120)
    method = rng.choice(["direct", "fft"])
    if rng.random() < 0.25:
        k = rng.choice([3, 5, 7, 9, 11])
        n, k = (1, _log_int(rng, 24, 288), _log_int(rng, 24, 288)), (1, k, k)
    else:
        a = rng.choice([2, 3, 3, 4, 5, 5, 6, 7])
        k = (rng.randint(1, a), a, a) if rng.random() < 0.3 else (a, a, a)
        e = _log_int(rng, 12, 96)
        n = (e, e, e) if rng.random() < 0.4 else tuple(_log_int(rng, max(8, e // 2), min(144, 2 * e)) for _ in range(3))
    s = rng.choice([2, 4]) if n[0] > 1 and max(k) <= 3 and rng.random() < 0.4 else 1
    if any(s * (b - 1) + 1 > a for a, b in zip(n, k)):
        return None
    c = _layer(f, fo, n, k, method, method == "fft" and rng.random() < 0.6, s)
    big = listed()
    if method == "direct":
        return c if work(c)["flops"] <= work(big[1])["flops"] else None
    # at most a quarter of the widest layer: an extent that the fast paths do not take costs more per voxel
    return c if f * fo * math.prod(n) <= 0.25 * 120 * 120 * 96 ** 3 else None


def _draw_net(rng, kind):
    family = rng.choice(["3d", "2d", "3d_sparse"])
    width = _log_int(rng, 6, 64)
    if kind == "train":
        patch = _log_int(rng, 16, 64) if family == "2d" else _log_int(rng, 3, 20)
        c = dict(kind=kind, family=family, width=width, patch=patch, replay=rng.random() < 0.4)
    else:
        patch = _log_int(rng, 32, 160) if family == "2d" else _log_int(rng, 10, 40)
        c = dict(kind=kind, family=family, width=width, patch=patch)
    return c if work(c)["flops"] <= 4e11 else None


def draw(rng):
    """One more case of the same ranges, costing no more than the widest layer above."""
    while True:
        kind = rng.choice(["layer"] * 5 + ["train"] * 3 + ["infer", "graph"])
        if kind == "layer":
            c = _draw_layer(rng)
        elif kind == "graph":
            c = dict(kind=kind, width=_log_int(rng, 4, 48), n=_log_int(rng, 14, 48))
        else:
            c = _draw_net(rng, kind)
        if c is not None:
            return c


# ------------------------------------------------------------------------------------------------- nets
def _net(case):
    """(layers, input shape) of a net family at the case's width and output patch."""
    w = case["width"]
    base = {"3d": synth.CONFIG3_LAYERS, "2d": synth.CONFIG2D_LAYERS, "3d_sparse": synth.CONFIG3_SPARSE_LAYERS}
    layers = [((l[0],) + tuple(w if m == synth.WIDTH else m for m in l[1:3]) + tuple(l[3:]) if l[0] == "conv" else l)
              for l in base[case["family"]]]
    # the output layer predicts labels in (0, 1); a rectifier there may die, and the whole gradient with it
    layers[-1] = ("transfer", "logistic")
    probe = (1, 1, 200, 200) if case["family"] == "2d" else (1, 200, 200, 200)
    shrink = 200 - synth.shapes(layers, probe)[-1][3]
    e = case["patch"] + shrink
    return layers, (1, 1, e, e) if case["family"] == "2d" else (1, e, e, e)


def _graph(case):
    return synth.multiscale_graph(width=case["width"], n=case["n"])


# -------------------------------------------------------------------------------------------- interface
def prepare(case, seed):
    if case["kind"] == "layer":
        n, k = (case["nz"], case["ny"], case["nx"]), (case["kz"], case["ky"], case["kx"])
        f, fo, s = case["f"], case["fo"], (case["s"],) * 3
        plan = znn.Plan(f, fo, n, k, case["method"], s)
        if case["memo"]:
            plan.enable_memo(DEV)
        gen = torch.Generator(device=DEV).manual_seed(seed)
        values = lambda shape, scale=1.0: (torch.rand(shape, generator=gen, device=DEV) * 2 - 1) * scale  # noqa: E731
        return {"case": case, "plan": plan, "x": values((f,) + n),
                "w": values((fo, f) + k, 1 / math.sqrt(f * math.prod(k))), "g": values((fo,) + plan.o),
                "out": torch.empty((fo,) + plan.o, device=DEV), "gin": torch.empty((f,) + n, device=DEV),
                "gw": torch.empty((fo, f) + k, device=DEV)}
    if case["kind"] == "graph":
        g = _graph(case)
        inputs, targets, params = synth.graph_tensors(g, seed)
        put = lambda d: {k: torch.from_numpy(v).to(DEV) for k, v in d.items()}  # noqa: E731
        eta = 0.01 / sum(t.size for t in targets.values())
        return {"case": case, "net": zgraph.GraphNet(g, params), "x": put(inputs), "t": put(targets), "eta": eta}
    layers, in_shape = _net(case)
    x, target, params = synth.net_tensors(layers, in_shape, seed)
    st = {"case": case, "net": znet.Net(layers, in_shape, params), "x": torch.from_numpy(x).to(DEV)}
    if case["kind"] == "train":
        st["t"], st["eta"] = torch.from_numpy(target).to(DEV), 0.01 / target.size
        if case["replay"]:
            st["replay"], st["recorded"] = st["net"].capture_round(st["x"], st["t"], st["eta"])
    return st


def run(state):
    case = state["case"]
    if case["kind"] == "layer":
        p, x, w, g, out, gin, gw = (state[k] for k in ("plan", "x", "w", "g", "out", "gin", "gw"))
        if case["memo"]:
            p.prepare_kernels(w)
            p.fwd(x, None, out)
            p.bwd(g, None, gin)
            p.wgrad_memo(gw)
        else:
            p.fwd(x, w, out)
            p.bwd(g, w, gin)
            p.wgrad(x, g, gw)
        return {"out": out, "gin": gin, "gw": gw}
    net = state["net"]
    if case["kind"] == "infer":
        return net.forward(state["x"])[0][-1]
    if case["kind"] == "graph":
        img, _, _, grads = net.train_round(state["x"], state["t"], state["eta"], "cross_entropy")
        return {"out": [img[n] for n in net.graph["outputs"]], "grads": grads, "params": net.params}
    if case["replay"]:
        state["replay"]()
        acts, _, _, grads = state["recorded"]
    else:
        acts, _, _, grads = net.train_round(state["x"], state["t"], state["eta"])
    return {"out": acts[-1], "grads": grads, "params": net.params}


def _smooth(n):
    while True:
        m = n
        for p in (2, 3, 5):
            while m % p == 0:
                m //= p
        if m == 1:
            return n
        n += 1


def _conv_flops(f, fo, n, k, s, passes, method=None):
    """FLOPs of a layer's passes (2 per multiply-add): by the direct method f f' n'^3 k^3 multiply-adds a
    pass; by the FFT method 2.5 N log2 N per real transform, one of every kernel and node and one product
    per edge and frequency for each pass; by the cheaper one where the library may choose."""
    o = [a - s * (b - 1) for a, b in zip(n, k)]
    direct = passes * 2.0 * f * fo * math.prod(o) * math.prod(k)
    N = [_smooth(a) for a in n]
    one = 2.5 * math.prod(N) * math.log2(max(2, math.prod(N)))
    kernels = f * fo * (2 if passes == 3 else 1)            # spectra of w, and the inverse for its gradient
    fft = one * (kernels + (f + fo) * min(2, passes)) + passes * 8.0 * f * fo * N[0] * N[1] * (N[2] // 2 + 1)
    return {"direct": direct, "fft": fft}.get(method, min(direct, fft))


def work(case):
    if case["kind"] == "layer":
        n, k = (case["nz"], case["ny"], case["nx"]), (case["kz"], case["ky"], case["kx"])
        f, fo, s = case["f"], case["fo"], case["s"]
        o = math.prod(a - s * (b - 1) for a, b in zip(n, k))
        values = 2 * f * math.prod(n) + 2 * fo * o + 2 * f * fo * math.prod(k)
        return {"bytes": 4.0 * values, "flops": _conv_flops(f, fo, n, k, s, 3, case["method"])}
    if case["kind"] == "graph":
        g = _graph(case)
        shape = synth.graph_shapes(g)
        edges = [(e[0], shape[e[2]], shape[e[3]], e[5] if e[0] == "conv" else None,
                  (e[6][0] if len(e) > 6 else 1) if e[0] == "conv" else 1) for e in g["edges"]]
        values = sum(math.prod(shape[n]) for n in g["inputs"]) + 2 * sum(math.prod(shape[n]) for n in g["outputs"])
    else:
        layers, in_shape = _net(case)
        shape = synth.shapes(layers, in_shape)
        edges = [(l[0], shape[i], shape[i + 1], l[3] if l[0] == "conv" else None,
                  (l[4][0] if len(l) > 4 else 1) if l[0] == "conv" else 1) for i, l in enumerate(layers)]
        values = math.prod(in_shape) + (2 if case["kind"] == "train" else 1) * math.prod(shape[-1])
        if case.get("family") == "2d":                      # tap spacing along z is no matter with one plane
            edges = [e[:4] + (1,) for e in edges]
    flops, passes = 0.0, 1 if case["kind"] == "infer" else 3
    for kind, a, b, k, s in edges:
        if kind == "conv":
            flops += _conv_flops(a[0], b[0], a[1:], k, s, passes)
            values += a[0] * b[0] * math.prod(k) * (1 if passes == 1 else 3)   # kernels; gradients, updated kernels
        else:
            flops += passes * math.prod(b)
    return {"bytes": 4.0 * values, "flops": flops}


def tolerance(case):
    # fp32 throughout: sums of up to some 40 000 products in another order, by either method
    if case["kind"] == "layer":
        return {"rel": 1e-5, "max": 2e-4}
    if case["kind"] == "infer":
        return {"rel": 2e-5, "max": 4e-4}
    # A rounding difference may open or close a rectifier at zero or pick the other voxel of a near-tie in a
    # max-filter window, which moves whole terms of the gradient sums.  The library's own two methods, each
    # right to 1e-6 per layer, differ by up to 1.8e-2 (max 7e-2) over 30 seeds of a net, typically 1e-6 to
    # 3e-3, and by up to 3e-4 (max 5e-3) on the graph, which has one filter on one of its branches.
    return {"rel": 2e-3, "max": 3e-2} if case["kind"] == "graph" else {"rel": 3e-2, "max": 0.3}
