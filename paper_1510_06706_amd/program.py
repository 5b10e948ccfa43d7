"""A round of a net as one native call (``znn_program_*``): the operations and their buffers.

``net`` and ``graph`` list the operations of a round once, with the buffers they work on; a run then
makes the tensors that the round returns, hands all pointers to the library in one call and launches
nothing itself.  Every arithmetic step runs in libznn's kernels.
"""
from __future__ import annotations

import ctypes
import math
import struct

from . import binding as znn
from .binding import TRANSFER_FNS

(CONV_FWD, CONV_BWD, CONV_WGRAD, TRANSFER_FWD, TRANSFER_BWD, BIAS_GRAD, FILTER_FWD, FILTER_BWD, POOL_FWD, POOL_BWD,
 LOSS_GRAD, NODE_SUM, UPDATE) = range(13)
LOSSES = {"square": 0, "cross_entropy": 1}
OP = struct.Struct("@22iP")         # the fields of binding.Op
assert OP.size == ctypes.sizeof(znn.Op)


class Program:
    """Buffers are numbers.  ``given`` ones are tensors of the caller, ``fresh`` ones are allocated by every
    run and returned, ``gradient`` ones likewise (all from one allocation), ``kept`` ones never leave the run: they
    and the scratch memory are allocated by every run and handed back behind it, so that a net holds nothing between
    its rounds, runs on any stream, and a recorded round owns what it works on."""

    # Bytes of kept buffers that have memory of their own.  Beyond it they take turns: the bias gradients then
    # come in a launch per layer instead of one (a few us of rounds that move more than this several times over).
    OWN_BYTES = 1 << 30

    def __init__(self, device, streams=1):
        self.device, self.streams = device, streams
        self.ops, self.plans = [], []
        self.shapes, self.kinds = [], []
        self._h = None

    # ------------------------------------------------------------ description
    def buffer(self, kind, shape, integer=False):
        self.shapes.append(tuple(shape))
        self.kinds.append((kind, integer))
        return len(self.kinds) - 1

    def add(self, kind, buf, stream=0, plan=None, fn="rectify", loss="square", maps=1, n=(1, 1, 1),
            window=(1, 1, 1), sparsity=(1, 1, 1)):
        """Adds an operation and returns it; what follows its result may still be attached to it."""
        op = dict(kind=kind, buf=list(buf) + [-1] * (8 - len(buf)), stream=stream, plan=plan, fn=TRANSFER_FNS[fn],
                  loss=LOSSES[loss], maps=maps, n=n, window=window, sparsity=sparsity)
        self.ops.append(op)
        return op

    @staticmethod
    def attach(op, fn, y=-1, bias=-1, gx=-1):
        """Lets `op` apply what follows it: a forward convolution the transfer function (bias, y), a loss gradient
        (gx) or a backward operation (y) the derivative of the edge below.  False if the operation cannot."""
        at = {CONV_FWD: ((3, bias), (4, y)), CONV_BWD: ((3, y),), FILTER_BWD: ((3, y),), POOL_BWD: ((3, y),),
              LOSS_GRAD: ((3, gx),), NODE_SUM: ((7, y),)}.get(op["kind"])
        if at is None or any(op["buf"][i] >= 0 for i, _ in at):
            return False
        for i, b in at:
            op["buf"][i] = b
        op["fn"] = TRANSFER_FNS[fn]
        return True

    def _take_turns(self):
        """Gives kept buffers whose uses do not overlap one number.  The library orders the operations by the
        buffers they name, so that this holds on several streams too."""
        first, last = {}, {}
        for i, d in enumerate(self.ops):
            for b in d["buf"]:
                if b >= 0 and self.kinds[b][0] == "kept":
                    first.setdefault(b, i)
                    last[b] = i
        number, free = {}, []                       # free: (last use, number) of the numbers in use so far
        for b in sorted(first, key=lambda b: first[b]):
            size = lambda f: math.prod(self.shapes[f[1]])  # noqa: E731
            idle = [f for f in free if f[0] < first[b]]
            # the largest idle one: its memory grows least
            f = max(idle, key=size) if idle else (-1, b)
            number[b] = f[1]
            if idle:
                free.remove(f)
                if math.prod(self.shapes[b]) > size(f):
                    self.shapes[f[1]] = self.shapes[b]
                self.kinds[b] = ("turn", f[1])
            free.append((last[b], f[1]))
        for d in self.ops:
            d["buf"] = [number.get(b, b) for b in d["buf"]]

    def build(self):
        n = len(self.kinds)
        if sum(4 * math.prod(s) for s, k in zip(self.shapes, self.kinds) if k[0] == "kept") > self.OWN_BYTES:
            self._take_turns()
        # The first round of a net pays for this: 242 us for the six-layer 3D net, and 367 with the table set field by field.
        table, known = [], set()
        for d in self.ops:
            plan = d["plan"]
            if plan is not None and id(plan) not in known:
                known.add(id(plan))
                self.plans.append((plan, plan.revision))
            table.append(OP.pack(d["kind"], d["stream"], d["fn"], d["loss"], d["maps"], *d["n"], *d["window"], *d["sparsity"],
                                 *d["buf"], 0 if plan is None else plan._h.value))
        ops = (znn.Op * len(table)).from_buffer_copy(b"".join(table))
        h = ctypes.c_void_p(0)
        znn._check(znn.lib().znn_program_create(ops, len(self.ops), n, self.streams, ctypes.byref(h)))
        self._h = h
        need = ctypes.c_size_t(0)
        znn._check(znn.lib().znn_program_scratch_bytes(h, ctypes.byref(need)))
        self.scratch_bytes = need.value
        up = lambda b: (b + 255) & ~255  # noqa: E731
        kept, slab = up(need.value), 0
        self._kept, self._grads, self._fresh = [], [], []
        for b, (kind, integer) in enumerate(self.kinds):
            size = 4 * math.prod(self.shapes[b])
            if kind == "kept":
                self._kept.append((b, kept))
                kept += up(size)
            elif kind == "gradient":
                self._grads.append((b, slab))
                slab += up(size)
            elif kind == "fresh":
                self._fresh.append((b, self.shapes[b], integer))
        at = dict(self._kept)
        self._kept += [(b, at[k[1]]) for b, k in enumerate(self.kinds) if k[0] == "turn"]
        self._kept_bytes, self._slab = kept, slab // 4
        return self

    def __del__(self):
        try:
            if self._h:
                znn.lib().znn_program_destroy(self._h)
                self._h = None
        except Exception:
            pass

    def current(self, plans):
        """Whether `plans`, in the order of their first operations, are those the program describes, as they were then."""
        return len(plans) == len(self.plans) and all(p is q and p.revision == r for p, (q, r) in zip(plans, self.plans))

    # ------------------------------------------------------------ runs
    def run(self, given, eta=0.0, streams=()):
        """given: {buffer: tensor}, checked by the caller.  Runs on the current stream (and `streams`, which
        it joins); returns {buffer: tensor} of the fresh and the gradient buffers."""
        import torch
        device = self.device
        buf, st = (ctypes.c_void_p * len(self.kinds))(), (ctypes.c_void_p * self.streams)()     # of this run alone
        base = None
        if self._kept_bytes:
            scratch = torch.empty(self._kept_bytes + 256, dtype=torch.uint8, device=device)
            base = (scratch.data_ptr() + 255) & ~255
        for b, at in self._kept:
            buf[b] = base + at
        for b, t in given.items():
            buf[b] = t.data_ptr()
        out = {}
        for b, shape, integer in self._fresh:
            t = out[b] = torch.empty(shape, dtype=torch.int32 if integer else torch.float32, device=device)
            buf[b] = t.data_ptr()
        if self._slab:
            slab = torch.empty(self._slab, dtype=torch.float32, device=device)
            for b, at in self._grads:
                buf[b] = slab.data_ptr() + at
        st[0] = torch.cuda.current_stream().cuda_stream
        for i, s in enumerate(streams):
            st[i + 1] = s.cuda_stream
        znn._check(znn.lib().znn_program_run(self._h, buf, base, self.scratch_bytes, eta, st))
        for b, at in self._grads:
            shape = self.shapes[b]
            out[b] = slab[at // 4:at // 4 + math.prod(shape)].view(shape)
        return out


def check_input(t, shape=None, count=None):
    """A tensor handed to a round: float32 values on the GPU, contiguous, of the shape (or at least the number of values) expected."""
    import torch
    if shape is not None:
        assert tuple(t.shape) == tuple(shape), t.shape
    if count is not None and t.numel() < count:
        raise ValueError("expected %d values, got %d" % (count, t.numel()))
    znn._ptr(t, torch.float32)
    return t


def check_parameter(t, key, shape):
    """The kernels ("w") of a layer, which the calls per layer take in their shape only, or its biases ("b")."""
    return check_input(t, shape) if key == "w" else check_input(t, count=math.prod(shape))
