"""One training round of a layered ConvNet driven through the C ABI (config-3 harness).

This module only sequences library calls (Section 3 of the paper: forward pass,
loss gradient, backward pass, gradients, update); every arithmetic step runs in
libznn's kernels.  The layer lists of the benchmark networks and their seeded
synthetic tensors live in ``synth``.
"""
from __future__ import annotations

import math

import numpy as np

from . import binding as znn
from . import program as zp
from .synth import ONES, _opt, shapes


class Net:
    """Device-side state of a layered net: plans per convolution, parameters as CUDA tensors.

    ``mode`` is "direct", "fft", "auto" (cached autotuner choice or cost model), a list with
    one entry per layer, or "tuned": every convolutional layer is timed as a whole round in
    the three strategies direct / FFT / FFT with memoized spectra (Section 4) and takes the
    fastest one whose buffers fit ``memory_budget`` bytes (per layer; None = no limit).  "fft_memo"
    (in a list) attaches memo buffers to the layer's plan, and rounds go layer by layer to leave the
    spectra there; rounds of tuned nets are programs, which memoize in their own memory.
    """

    def __init__(self, layers, in_shape, params, mode="auto", device="cuda:0", memory_budget=None):
        import torch
        self.layers = list(layers)
        self.shapes = shapes(layers, in_shape)
        self.device = device
        self.params = [None if p is None else {k: torch.from_numpy(np.ascontiguousarray(v)).to(device)
                                               for k, v in p.items()} for p in params]
        self.plans = []
        self.strategy = [None] * len(self.layers)
        self.tuning = {}
        for l, spec in enumerate(self.layers):
            if spec[0] == "conv":
                m = mode[l] if isinstance(mode, (list, tuple)) else mode
                sp = _opt(spec, 4, ONES)
                if m == "tuned":
                    m, ms, nbytes = znn.autotune_round(spec[1], spec[2], self.shapes[l][1:], spec[3],
                                                       memory_budget, sp, device)
                    self.tuning[l] = (m, ms, nbytes)
                    spare = None if memory_budget is None else max(0, memory_budget - nbytes[m])
                else:
                    spare = None
                plan = znn.Plan(spec[1], spec[2], self.shapes[l][1:], spec[3], "fft" if m == "fft_memo" else m, sp)
                if m == "fft_memo" and l not in self.tuning:
                    plan.enable_memo(device)
                elif spare is not None:         # the budget holds for rounds as one program as well
                    # which do the memoizing of a tuned net: its plans get no buffers beside theirs
                    plan.set_round_memory(spare + (plan.spectra_bytes() + plan.memo_bytes() if m == "fft_memo" else 0))
                self.strategy[l] = m
                self.plans.append(plan)
            else:
                self.plans.append(None)
        self._programs = {}

    @property
    def _by_layer(self):
        """Whether rounds go layer by layer: plans that were given memo buffers leave their spectra there, and in a
        program a plan stands for one layer, where the caller may have set one for several of a shape."""
        plans = [p for p in self.plans if p is not None]
        return any(p._memo is not None for p in plans) or len({id(p) for p in plans}) < len(plans)

    def _memoized(self, l):
        """Whether the calls of layer l, one by one, leave their spectra in its plan."""
        return self.strategy[l] == "fft_memo" and self.plans[l]._memo is not None

    def modes(self):
        return [None if p is None else p.mode for p in self.plans]

    # ------------------------------------------------------------ rounds as one native call
    def _program(self, loss):
        """The forward pass (loss None) or a whole training round as a program on the calling stream (kernel gradients
        on a second stream gained nothing: 410 against 422 us a round of the six-layer 3D net, 40 us slower replayed)."""
        if loss in self._programs and self._programs[loss][0].current([p for p in self.plans if p is not None]):
            return self._programs[loss]
        P = zp.Program(self.device)
        L, shape = self.layers, self.shapes
        given = {(0, "x"): P.buffer("given", shape[0])}
        for l, spec in enumerate(L):
            if spec[0] == "conv":
                given[l, "w"] = P.buffer("given", (spec[2], spec[1]) + tuple(spec[3]))
            elif spec[0] == "transfer":
                given[l, "b"] = P.buffer("given", shape[l][:1])
        act, aux, conv = [given[0, "x"]], [None] * len(L), None
        for l, spec in enumerate(L):
            kind, y = spec[0], P.buffer("fresh", shape[l + 1])
            if kind == "conv":
                conv = P.add(zp.CONV_FWD, (act[-1], given[l, "w"], y), plan=self.plans[l])
            elif kind == "transfer":
                fn = _opt(spec, 1, "rectify")
                if conv is None or not P.attach(conv, fn, y, given[l, "b"]):
                    P.add(zp.TRANSFER_FWD, (act[-1], given[l, "b"], y), fn=fn, maps=shape[l][0], n=shape[l][1:])
            else:
                aux[l] = P.buffer("fresh", shape[l + 1], True)
                P.add(zp.FILTER_FWD if kind == "maxfilter" else zp.POOL_FWD, (act[-1], y, aux[l]), maps=shape[l][0],
                      n=shape[l][1:], window=spec[1], sparsity=_opt(spec, 2, ONES) if kind == "maxfilter" else ONES)
            if kind != "conv":
                conv = None
            act.append(y)
        grads, gout, target = [None] * len(L), None, None
        if loss is not None:
            target, gout = P.buffer("given", shape[-1]), P.buffer("fresh", shape[-1])
            g, op = gout, P.add(zp.LOSS_GRAD, (act[-1], target, gout), loss=loss, maps=shape[-1][0], n=shape[-1][1:])
            for l in range(len(L) - 1, -1, -1):
                spec, kind = L[l], L[l][0]
                below = lambda: P.buffer("kept", shape[l])  # noqa: B023,E731
                how = dict(maps=shape[l][0], n=shape[l][1:])
                if kind == "transfer":
                    # the operation that completed g applies the derivative itself where it can
                    fn = _opt(spec, 1, "rectify")
                    if op is None or op["kind"] == zp.LOSS_GRAD or not P.attach(op, fn, act[l + 1]):
                        h = below()
                        if op is None or not P.attach(op, fn, gx=h):
                            P.add(zp.TRANSFER_BWD, (g, act[l + 1], h), fn=fn, **how)
                        g = h
                    grads[l] = {"b": P.buffer("gradient", (shape[l][0],))}
                    P.add(zp.BIAS_GRAD, (g, grads[l]["b"]), **how)
                    op = None
                elif kind == "conv":
                    grads[l] = {"w": P.buffer("gradient", P.shapes[given[l, "w"]])}
                    ready = g
                    if l > 0:
                        g = below()
                        op = P.add(zp.CONV_BWD, (ready, given[l, "w"], g), plan=self.plans[l])
                    P.add(zp.CONV_WGRAD, (act[l], ready, grads[l]["w"]), plan=self.plans[l])
                elif l > 0:
                    h = below()
                    op = P.add(zp.FILTER_BWD if kind == "maxfilter" else zp.POOL_BWD, (g, aux[l], h), window=spec[1],
                               sparsity=_opt(spec, 2, ONES) if kind == "maxfilter" else ONES, **how)
                    g = h
            for l, d in enumerate(grads):
                for k in d or ():
                    P.add(zp.UPDATE, (d[k], given[l, k]), n=(1, 1, math.prod(P.shapes[d[k]])))
        self._programs[loss] = P.build(), given, act, aux, target, gout, grads
        return self._programs[loss]

    def _run(self, loss, x, target=None, eta=0.0):
        P, given, act, aux, t, gout, grads = self._program(loss)
        tensors = {given[0, "x"]: zp.check_input(x, self.shapes[0])}
        for (l, k), b in given.items():
            if k != "x":
                tensors[b] = zp.check_parameter(self.params[l][k], k, P.shapes[b])
        if loss is not None:
            tensors[t] = zp.check_input(target, count=math.prod(self.shapes[-1]))
        out = P.run(tensors, float(eta))
        return ([x] + [out[b] for b in act[1:]], [None if b is None else out[b] for b in aux],
                None if gout is None else out[gout],
                [None if d is None else {k: out[b] for k, b in d.items()} for d in grads])

    def forward(self, x):
        # without convolutions, inputs of any extent pass
        if self._by_layer or tuple(x.shape) != tuple(self.shapes[0]):
            return self._forward_by_layer(x)
        return self._run(None, x)[:2]

    def _forward_by_layer(self, x):
        """One library call per layer: what plans with memoized spectra of their own need before ``backward``."""
        acts, aux = [x], [None] * len(self.layers)
        for l, spec in enumerate(self.layers):
            a = acts[-1]
            if spec[0] == "conv" and self._memoized(l):
                self.plans[l].prepare_kernels(self.params[l]["w"])      # once per round: w changes every update
                y = self.plans[l].fwd(a, None)
            elif spec[0] == "conv":
                y = self.plans[l].fwd(a, self.params[l]["w"])
            elif spec[0] == "transfer":
                y = znn.transfer_fwd(a, self.params[l]["b"], _opt(spec, 1, "rectify"))
            elif spec[0] == "maxfilter":
                y, aux[l] = znn.maxfilter3d_fwd(a, spec[1], _opt(spec, 2, ONES))
            else:
                y, aux[l] = znn.maxpool3d_fwd(a, spec[1])
            acts.append(y)
        return acts, aux

    def backward(self, acts, aux, gout, record=None):
        """`record`, if a list, receives (layer, gradient arriving at that layer's output)."""
        grads = [None] * len(self.layers)
        g = gout
        for l in range(len(self.layers) - 1, -1, -1):
            spec = self.layers[l]
            if record is not None:
                record.append((l, g))
            if spec[0] == "conv" and self._memoized(l) and l > 0:
                # backward first: it leaves the spectra of g next to those of the forward input
                g = self.plans[l].bwd(g, None)
                grads[l] = {"w": self.plans[l].wgrad_memo(device=self.device)}
            elif spec[0] == "conv":
                grads[l] = {"w": self.plans[l].wgrad(acts[l], g)}
                g = self.plans[l].bwd(g, self.params[l]["w"]) if l > 0 else None
            elif spec[0] == "transfer":
                g = znn.transfer_bwd(g, acts[l + 1], _opt(spec, 1, "rectify"))
                grads[l] = {"b": znn.bias_grad(g)}
            elif spec[0] == "maxfilter":
                g = znn.maxfilter3d_bwd(g, aux[l], self.shapes[l][1:], spec[1], _opt(spec, 2, ONES))
            else:
                g = znn.maxpool3d_bwd(g, aux[l], self.shapes[l][1:], spec[1])
        return grads

    def train_round(self, x, target, eta, record=None, loss="square"):
        if loss not in zp.LOSSES:
            raise ValueError(loss)
        if record is None and not self._by_layer:
            return self._run(loss, x, target, eta)
        acts, aux = self._forward_by_layer(x)
        gout = znn.loss_grad(acts[-1], target, loss)
        grads = self.backward(acts, aux, gout, record)
        for p, g in zip(self.params, grads):
            if p is not None:
                for k in p:
                    znn.sgd_update(p[k], g[k], eta)
        return acts, aux, gout, grads

    def capture_round(self, x, target, eta, loss="square"):
        """Records one training round (all library launches on the current HIP stream, no host
        synchronisation, no memset) into a HIP graph and returns ``(replay, outputs)``:
        ``replay()`` re-runs the round on the same buffers - new inputs are copied into ``x`` and
        ``target`` in place, the parameters are updated in place - without per-launch host cost;
        ``outputs = (acts, aux, gout, grads)`` are the graph's own output tensors.  Workspaces and
        resident spectra are allocated by a warm-up round before the capture."""
        import torch
        side = torch.cuda.Stream(device=self.device)
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):       # warm-up outside the graph: plans grow their workspaces
            saved = [None if p is None else {k: v.clone() for k, v in p.items()} for p in self.params]
            self.train_round(x, target, eta, loss=loss)
            for p, q in zip(self.params, saved):
                if p is not None:
                    for k in p:
                        p[k].copy_(q[k])
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            outputs = self.train_round(x, target, eta, loss=loss)
        return graph.replay, outputs
