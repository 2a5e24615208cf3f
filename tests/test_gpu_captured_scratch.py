"""Graphs that a caller captured from the library's calls stay valid when later
calls on the stream need more scratch: what they were captured with is kept.
Between capture and replay the scratch grows and other allocations are made and
filled. Every replay is checked against the oracle, exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import (assert_same, dev, log, make_fill, oracle_result, pad_stride, poison, poison_out,  # noqa: E402
                      poison_q, poison_z)
from test_gpu_compress import check, packed_out, rows  # noqa: E402

PARAMS = {"threshold": -200, "pre": 8, "post": 24, "ped_samples": 100}


def _raw(rng, N, C=2):
    x = rng.integers(995, 1006, size=(C, N)).astype(np.int16)
    x[0, rng.integers(0, N, N // 100 + 1)] -= 500
    return pad_stride(x)


class Chop:
    """n fills through the batch call, or one through the single-fill call."""

    def __init__(self, rng, n, N, single=False):
        xs = [_raw(rng, N + i) for i in range(n)]
        self.fills = [make_fill(dev(x), N + i, PARAMS) for i, x in enumerate(xs)]
        self.refs = [oracle_result(x, N + i, PARAMS) for i, x in enumerate(xs)]
        self.outs = [daq.alloc_out(f) for f in self.fills]
        self.single = single

    def call(self, ctx):
        if self.single:
            ctx.daq_chop_fill(self.fills[0], self.outs[0])
        else:
            ctx.daq_process_batch(self.fills, self.outs)

    def check(self, what):
        torch.cuda.synchronize()
        for i, (o, r) in enumerate(zip(self.outs, self.refs)):
            assert_same(o, r, ctx="%s fill %d" % (what, i))
            poison_out(o)
        torch.cuda.synchronize()


class QMethod:
    def __init__(self, rng, n, N, C=2):
        xs = [_raw(rng, N, C) for _ in range(n)]
        self.fills = [make_fill(dev(x), N, PARAMS) for x in xs]
        self.refs = [oracle.qmethod(x, N)[1] for x in xs]
        self.outs = [daq.alloc_q_out(f, acc=False) for f in self.fills]
        for q in self.outs:
            q.ped = None  # the pedestals then go to the stream's scratch

    def call(self, ctx):
        ctx.daq_qmethod_batch(self.fills, self.outs)

    def check(self, what):
        torch.cuda.synchronize()
        for q, r in zip(self.outs, self.refs):
            np.testing.assert_array_equal(q.qsum.cpu().numpy()[:len(r)], r, err_msg=what)
            poison_q(q)
        torch.cuda.synchronize()


class Compress:
    def __init__(self, rng, n, L, C):
        self.xs, self.L = [rows(i, C, L, "noise") for i in range(n)], L
        self.ins = [packed_out(x, L) for x in self.xs]
        self.outs = [daq.alloc_z_out(C, o.out.shape[1], device="cuda") for o in self.ins]

    def call(self, ctx):
        ctx.daq_compress_batch(self.ins, self.outs)

    def check(self, what):
        torch.cuda.synchronize()
        for z, x in zip(self.outs, self.xs):
            check(z, x, self.L, what)
            poison_z(z)
        torch.cuda.synchronize()


KINDS = {
    "single": (lambda r: Chop(r, 1, 5000, True), lambda r: Chop(r, 1, 3_000_000, True)),
    "batch 3": (lambda r: Chop(r, 3, 3000), lambda r: Chop(r, 120, 40_000)),
    "batch 20": (lambda r: Chop(r, 20, 1500), lambda r: Chop(r, 200, 40_000)),
    "qmethod": (lambda r: QMethod(r, 2, 5000), lambda r: QMethod(r, 100, 2000, 70)),
    "compress": (lambda r: Compress(r, 2, 5000, 3), lambda r: Compress(r, 1, 60_000, 54)),
}


@pytest.mark.parametrize("kind", list(KINDS))
def test_a_captured_call_outlives_the_growth_of_its_scratch(kind):
    rng = np.random.default_rng(len(kind))
    small, large = (make(rng) for make in KINDS[kind])
    with daq.Context(0) as ctx:
        ctx.set_schedule(512, 8, 5, 0)  # launched plainly, whatever the environment says
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            small.call(ctx)  # the scratch of a small call
        small.check("plain")
        log("capture " + kind)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            small.call(ctx)
        with torch.cuda.stream(s):
            g.replay()
        small.check("replay before")
        for k in range(3):
            with torch.cuda.stream(s):
                large.call(ctx)  # grows the scratch the first time
            large.check("large %d" % k)
            taken = [poison(torch.empty(1 << b, dtype=torch.uint8, device="cuda")) for b in range(12, 25)]
            log("%s replay %d" % (kind, k))
            with torch.cuda.stream(s):
                g.replay()
            small.check("replay %d" % k)
            with torch.cuda.stream(s):
                small.call(ctx)
            small.check("plain %d" % k)
            for t in taken:
                assert bool((t == 0x5A).all())
        del g
