"""One training round on a general computation graph, run as a multi-stream launch DAG.

Section 2 of the paper: nodes hold images, edges are convolutions, max-filters, max-pools
or transfer functions, and a node's image is the sum of the edges converging on it; the
graph need not be layered (branches with different sparsity may fan out of a node and
converge again: multi-scale nets).  Section 3: the backward graph is the same graph
reversed, a node's backward image being the sum over its outgoing edges.

The paper's CPU design runs the edges as tasks on worker threads.  On the GPU the same
dependency structure becomes streams and events: every edge is launched on one of a few
HIP streams, so independent branches overlap on the device, and the kernel-gradient of an edge
runs on another stream than its backward image (they only share inputs).  Sums at nodes are
taken in the fixed order of the edge list (every converging edge writes its own buffer), so
results do not depend on which stream finished first.

A round (``GraphNet.train_round``) is one native program: the library orders its operations by
the buffers they use, with events of its own, forks every stream from the calling one and joins
it again.  ``GraphNet.forward`` and ``backward`` run the passes edge by edge, one library call
each, for callers that want node images or gradients without a round.

This module only sequences library calls; every arithmetic step runs in libznn's kernels.
The graph format is the one of ``synth.graph_shapes``.
"""
from __future__ import annotations

import math

import numpy as np

from . import binding as znn
from . import program as zp
from .synth import ONES, _opt, graph_shapes


def edge_order(graph):
    """Edge list reordered so that all edges into a node precede every edge out of it."""
    edges = list(graph["edges"])
    remaining_in = {}
    for e in edges:
        remaining_in[e[3]] = remaining_in.get(e[3], 0) + 1
    ready = set(graph["inputs"])
    out, pending = [], edges
    while pending:
        rest = []
        for e in pending:
            if e[2] in ready:
                out.append(e)
                remaining_in[e[3]] -= 1
                if remaining_in[e[3]] == 0:
                    ready.add(e[3])
            else:
                rest.append(e)
        if len(rest) == len(pending):
            raise ValueError("graph has a cycle or an edge whose source is never produced")
        pending = rest
    return out


class GraphNet:
    """Device-side state of a computation graph: plans per convolution edge, parameters as
    CUDA tensors, a pool of HIP streams (all at the default priority).

    Edge by edge, ``forward`` and ``backward`` wait on pooled events that were first recorded by an
    earlier pass, and join their side streams only through the events of later edges: they run eagerly
    only.  Every tensor of a pass stays referenced until the pass has joined the calling stream, and the
    next pass starts from events recorded after that join, so memory handed back to the allocator is never
    reused while another stream still reads it.

    ``streams`` is the number of side streams.  None stands for four, of which a round uses all or, where it is
    small, none; a number is kept to by every round."""

    # Multiply-adds of a round's convolutions by the direct method, times two, from which on several streams may be the faster ones.  Multi-scale nets, us a round
    # on several streams and on one: width 8, 20^3 443 and 164; 16, 40^3 (6e9) 483 and 311; 32, 40^3 (2.4e10) 543 and 510; 40, 36^3 (2.5e10) 551 and 555;
    # 36, 40^3 (3e10) 651 and 651; 44, 40^3 (4.4e10) 757 and 761; 48, 40^3 (5.2e10) 766 and 793; 48, 48^3 (1e11) 1465 and 1519; all by the FFT method 24, 48^3
    # (2.5e10) 810 and 786; 40, 40^3 (3.6e10) 818 and 861.  Independent branches that never meet gain less by streams, as each edge brings its waits:
    # two to eight, two to four layers deep, 2D and 3D, either method (1e8 to 5.5e10), one took 0.35 to 0.98 of the time of several.
    SEVERAL_STREAMS = 3e10

    def __init__(self, graph, params, mode="auto", device="cuda:0", streams=None):
        import torch
        self.graph = graph
        self.device = device
        self.shapes = graph_shapes(graph)
        self.edges = edge_order(graph)
        self.params = {n: {k: torch.from_numpy(np.ascontiguousarray(v)).to(device) for k, v in p.items()}
                       for n, p in params.items()}
        self.streams = [torch.cuda.Stream(device=device) for _ in range(4 if streams is None else max(1, int(streams)))]
        self._given_streams = streams is not None
        self._programs = {}
        self._events, self._next_event = [], 0      # events are reused from round to round
        self.incoming, self.outgoing = {}, {}
        for e in self.edges:
            self.incoming.setdefault(e[3], []).append(e[1])
            self.outgoing.setdefault(e[2], []).append(e[1])
        for n in self.shapes:
            if n not in graph["outputs"] and n not in self.outgoing:
                raise ValueError("node %r reaches no output" % (n,))
        # two plans per convolution edge: edge by edge, forward and backward image run on one stream and the
        # kernel gradient on another, each with its own workspace (programs need one)
        self.plans, self.plans_w = {}, {}
        for e in self.edges:
            if e[0] == "conv":
                f, n = self.shapes[e[2]][0], self.shapes[e[2]][1:]
                m = mode[e[1]] if isinstance(mode, dict) else mode
                self.plans[e[1]] = znn.Plan(f, e[4], n, e[5], m, _opt(e, 6, ONES))
                self.plans_w[e[1]] = znn.Plan(f, e[4], n, e[5], self.plans[e[1]].mode, _opt(e, 6, ONES))

    def modes(self):
        return {n: p.mode for n, p in self.plans.items()}

    # ------------------------------------------------------------ helpers
    def _stream_of(self, i):
        return self.streams[i % len(self.streams)]

    def _event(self, stream):
        """An event from the pool, recorded on `stream`."""
        import torch
        if self._next_event == len(self._events):
            self._events.append(torch.cuda.Event())
        ev = self._events[self._next_event]
        self._next_event += 1
        ev.record(stream)
        return ev

    @staticmethod
    def _sum_in_order(parts, order, events, stream):
        """parts[name] are separate buffers; adds them in `order` on `stream` after their events."""
        import torch
        for name in order:
            stream.wait_event(events[name])
        total = parts[order[0]]
        if len(order) > 1:
            with torch.cuda.stream(stream):
                total = total.clone()   # the first part stays intact (it may be an edge's kept output)
        for name in order[1:]:
            znn.accumulate(total, parts[name], stream=stream)
        return total

    # ------------------------------------------------------------ passes
    def forward(self, inputs):
        """inputs: {node: CUDA tensor}.  Returns (node images, per-edge aux, node events)."""
        import torch
        main = torch.cuda.current_stream()
        self._next_event = 0
        img, aux, ready = dict(inputs), {}, {}
        first = self._event(main)
        for n in inputs:
            ready[n] = first
        parts, part_ev = {}, {}
        for i, e in enumerate(self.edges):
            kind, name, src, dst = e[:4]
            s = self._stream_of(i)
            s.wait_event(ready[src])
            a = img[src]
            if kind == "conv":
                y = self.plans[name].fwd(a, self.params[name]["w"], stream=s)
            elif kind == "transfer":
                y = aux[name] = znn.transfer_fwd(a, self.params[name]["b"], _opt(e, 4, "rectify"), stream=s)
            elif kind == "maxfilter":
                y, aux[name] = znn.maxfilter3d_fwd(a, e[4], _opt(e, 5, ONES), stream=s)
            else:
                y, aux[name] = znn.maxpool3d_fwd(a, e[4], stream=s)
            parts.setdefault(dst, {})[name] = y
            part_ev[name] = self._event(s)
            if len(parts[dst]) == len(self.incoming[dst]):       # last edge into dst: take the sum
                img[dst] = self._sum_in_order(parts[dst], self.incoming[dst], part_ev, s)
                ready[dst] = part_ev[name] if len(self.incoming[dst]) == 1 else self._event(s)
        for n in self.graph["outputs"]:
            main.wait_event(ready[n])
        return img, aux, ready

    def backward(self, img, aux, gout):
        """gout: {output node: d loss / d image} (valid on the current stream).  Returns
        (parameter gradients per edge name, backward images per node)."""
        import torch
        main = torch.cuda.current_stream()
        back, ready, grads, grad_ev = {}, {}, {}, []
        parts, part_ev = {}, {}
        start = self._event(main)     # forward images and gout are complete at this point of `main`
        for n, g in gout.items():
            parts.setdefault(n, {})["loss"] = g
            part_ev["loss:" + n] = start

        def finish(node, stream):
            order = ["loss"] * (node in gout) + list(reversed(self.outgoing.get(node, [])))
            evs = {k: part_ev["loss:" + node] if k == "loss" else part_ev[k] for k in order}
            back[node] = self._sum_in_order(parts[node], order, evs, stream)
            ready[node] = self._event(stream)

        for n in gout:
            if n not in self.outgoing:
                finish(n, main)
        for i, e in enumerate(reversed(self.edges)):
            kind, name, src, dst = e[:4]
            s = self._stream_of(i)
            s.wait_event(ready[dst])
            s.wait_event(start)
            g = back[dst]
            if kind == "conv":
                sw = self._stream_of(i + 1 + len(self.streams) // 2)
                sw.wait_event(ready[dst])
                sw.wait_event(start)
                grads[name] = {"w": self.plans_w[name].wgrad(img[src], g, stream=sw)}
                grad_ev.append(self._event(sw))
                gs = None if src in self.graph["inputs"] else self.plans[name].bwd(g, self.params[name]["w"], stream=s)
            elif kind == "transfer":
                gs = znn.transfer_bwd(g, aux[name], _opt(e, 4, "rectify"), stream=s)
                grads[name] = {"b": znn.bias_grad(gs, stream=s)}
            elif kind == "maxfilter":
                gs = znn.maxfilter3d_bwd(g, aux[name], self.shapes[src][1:], e[4], _opt(e, 5, ONES), stream=s)
            else:
                gs = znn.maxpool3d_bwd(g, aux[name], self.shapes[src][1:], e[4], stream=s)
            ev = self._event(s)
            grad_ev.append(ev)
            if gs is None:
                continue
            parts.setdefault(src, {})[name] = gs
            part_ev[name] = ev
            if len(parts[src]) == len(self.outgoing[src]) + (src in gout):
                finish(src, s)
        for ev in grad_ev:
            main.wait_event(ev)
        return grads, back

    # ------------------------------------------------------------ rounds as one native call
    def _side_streams(self):
        """The streams of a round.  Its waits between streams take 5 to 12 us each, which only long edges pay for."""
        if self._given_streams:
            return self.streams
        flops = sum(6.0 * self.shapes[e[2]][0] * e[4] * math.prod(self.shapes[e[3]][1:]) * math.prod(e[5])
                    for e in self.edges if e[0] == "conv")
        return self.streams if flops >= self.SEVERAL_STREAMS else []

    def _build(self, loss):
        """A training round as a program: edge i runs on stream 1 + i mod (number of streams), kernel gradients half
        the streams further on, sums at a node on the stream of the last edge into it; the loss gradients and
        the update run on the calling stream, and all of a small round does.  Where an edge alone fills a node, what follows the node is
        applied by that edge's operation."""
        g, shape, E = self.graph, self.shapes, self.edges
        side = self._side_streams()
        P = zp.Program(self.device, 1 + len(side))
        stream = lambda i: 1 + i % len(side) if side else 0  # noqa: E731
        given = {(n, "x"): P.buffer("given", shape[n]) for n in g["inputs"]}
        for e in E:
            if e[0] == "conv":
                given[e[1], "w"] = P.buffer("given", (e[4], shape[e[2]][0]) + tuple(e[5]))
            elif e[0] == "transfer":
                given[e[1], "b"] = P.buffer("given", shape[e[2]][:1])
        by_name = {e[1]: e for e in E}

        def parts_sum(out, parts, at, dims):
            """Operation(s) that add `parts` in order into buffer `out`; the last one."""
            while True:
                op = P.add(zp.NODE_SUM, [out] + parts[:6], stream=at, maps=dims[0], n=dims[1:])
                if len(parts) <= 6:
                    return op
                parts = [out] + parts[6:]

        # forward: img[n] is node n's image, aux[e] what the backward edge reads
        img, aux, part = {n: given[n, "x"] for n in g["inputs"]}, {}, {}
        alone = lambda n: len(self.incoming[n]) == 1  # noqa: E731
        for i, e in enumerate(E):
            kind, name, src, dst = e[:4]
            how = dict(stream=stream(i), maps=shape[src][0], n=shape[src][1:])
            if name not in part:                # a transfer edge may have been taken over by the convolution before it
                y = part[name] = P.buffer("fresh" if alone(dst) or kind == "transfer" else "kept", shape[dst])
                if kind == "conv":
                    op = P.add(zp.CONV_FWD, (img[src], given[name, "w"], y), stream=stream(i), plan=self.plans[name])
                    then = next((by_name[n] for n in self.outgoing.get(dst, ()) if by_name[n][0] == "transfer"), None)
                    if alone(dst) and then is not None:
                        aux[then[1]] = part[then[1]] = P.buffer("fresh", shape[then[3]])
                        P.attach(op, _opt(then, 4, "rectify"), part[then[1]], given[then[1], "b"])
                elif kind == "transfer":
                    aux[name] = y
                    P.add(zp.TRANSFER_FWD, (img[src], given[name, "b"], y), fn=_opt(e, 4, "rectify"), **how)
                else:
                    aux[name] = P.buffer("fresh", shape[dst], True)
                    P.add(zp.FILTER_FWD if kind == "maxfilter" else zp.POOL_FWD, (img[src], y, aux[name]), window=e[4],
                          sparsity=_opt(e, 5, ONES) if kind == "maxfilter" else ONES, **how)
            if all(n in part for n in self.incoming[dst]) and dst not in img:
                if alone(dst):
                    img[dst] = part[name]
                else:
                    img[dst] = P.buffer("fresh", shape[dst])
                    parts_sum(img[dst], [part[n] for n in self.incoming[dst]], stream(i), shape[dst])

        # backward: back[n] is node n's backward image, `below` the transfer edge whose derivative it already holds
        gout, targets, back, below, gpart, grads = {}, {}, {}, {}, {}, {}
        outgoing = lambda n: list(reversed(self.outgoing.get(n, [])))  # noqa: E731

        def finish(node, at):
            order = ["loss"] * (node in gout) + outgoing(node)
            buf, op = gpart[node][order[0]]
            if len(order) > 1:
                buf = P.buffer("kept", shape[node])
                op = parts_sum(buf, [gpart[node][k][0] for k in order], at, shape[node])
            # the only edge into the node is a transfer function: its derivative with the sum
            e = by_name[self.incoming[node][0]] if alone(node) else None
            if e is not None and e[0] == "transfer":
                if op["kind"] == zp.LOSS_GRAD:
                    gx = P.buffer("kept", shape[node])
                    P.attach(op, _opt(e, 4, "rectify"), gx=gx)
                    buf, below[node] = gx, e[1]
                elif P.attach(op, _opt(e, 4, "rectify"), aux[e[1]]):
                    below[node] = e[1]
            back[node] = (buf, op)

        for n in g["outputs"]:
            gout[n], targets[n] = P.buffer("fresh", shape[n]), P.buffer("given", shape[n])
            op = P.add(zp.LOSS_GRAD, (img[n], targets[n], gout[n]), loss=loss, maps=shape[n][0], n=shape[n][1:])
            gpart.setdefault(n, {})["loss"] = (gout[n], op)
            if n not in self.outgoing:
                finish(n, 0)
        for i, e in enumerate(reversed(E)):
            kind, name, src, dst = e[:4]
            s, (b, op) = stream(i), back[dst]
            how = dict(stream=s, maps=shape[src][0], n=shape[src][1:])
            needed = src not in g["inputs"]
            gs = None
            if kind == "conv":
                grads[name] = {"w": P.buffer("gradient", P.shapes[given[name, "w"]])}
                if needed:
                    gs = P.buffer("kept", shape[src])
                    gop = P.add(zp.CONV_BWD, (b, given[name, "w"], gs), stream=s, plan=self.plans[name])
                P.add(zp.CONV_WGRAD, (img[src], b, grads[name]["w"]), stream=stream(i + 1 + len(side) // 2),
                      plan=self.plans[name])
            elif kind == "transfer":
                if below.get(dst) == name:
                    gs, gop = b, dict(op, kind=None)
                else:
                    gs = P.buffer("kept", shape[src])
                    gop = P.add(zp.TRANSFER_BWD, (b, aux[name], gs), fn=_opt(e, 4, "rectify"), **how)
                grads[name] = {"b": P.buffer("gradient", (shape[src][0],))}
                P.add(zp.BIAS_GRAD, (gs, grads[name]["b"]), **how)
            elif needed:
                gs = P.buffer("kept", shape[src])
                gop = P.add(zp.FILTER_BWD if kind == "maxfilter" else zp.POOL_BWD, (b, aux[name], gs), window=e[4],
                            sparsity=_opt(e, 5, ONES) if kind == "maxfilter" else ONES, **how)
            if gs is None or not needed:
                continue
            gpart.setdefault(src, {})[name] = (gs, gop)
            if len(gpart[src]) == len(self.outgoing[src]) + (src in gout):
                finish(src, s)
        for n, d in grads.items():
            for k in d:
                P.add(zp.UPDATE, (d[k], given[n, k]), n=(1, 1, math.prod(P.shapes[d[k]])))
        return P.build(), given, targets, img, aux, gout, grads

    def train_round(self, inputs, targets, eta, loss="square"):
        """Forward, loss gradient at every output node, backward, update (Algorithm 3).  The
        update runs after every stream has joined: kernels are read by the backward edges."""
        if loss not in zp.LOSSES:
            raise ValueError(loss)
        if loss not in self._programs or not self._programs[loss][0].current(list(self.plans.values())):
            self._programs[loss] = self._build(loss)
        P, given, target, img, aux, gout, grads = self._programs[loss]
        tensors = {given[n, "x"]: zp.check_input(inputs[n], self.shapes[n]) for n in self.graph["inputs"]}
        for (n, k), b in given.items():
            if k != "x":
                tensors[b] = zp.check_parameter(self.params[n][k], k, P.shapes[b])
        for n, b in target.items():
            tensors[b] = zp.check_input(targets[n], count=math.prod(self.shapes[n]))
        out = P.run(tensors, float(eta), self.streams[:P.streams - 1])
        out.update({given[n, "x"]: inputs[n] for n in self.graph["inputs"]})
        return ({n: out[b] for n, b in img.items()}, {n: out[b] for n, b in aux.items()}, {n: out[b] for n, b in gout.items()},
                {n: {k: out[b] for k, b in d.items()} for n, d in grads.items()})
