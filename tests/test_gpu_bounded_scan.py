"""Schedules that bound the split variant's scan to a few work-groups per CU, in
launches on both sides of the length (eight rounds of tiles) from which they do.
Against the oracle, exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import assert_same, dev, log, make_fill, oracle_many, pad_stride, poison_out  # noqa: E402

TILE = 512
PARAMS = {"threshold": -200, "pre": 8, "post": 24, "ped_samples": 100}


def _fill(rng, C, N):
    x = rng.integers(995, 1006, size=(C, N)).astype(np.int16)
    x[C - 1, rng.integers(0, N, N // 1000 + 2)] -= 500
    return pad_stride(x)


def _check(ctx, C, ns, what, seed=1):
    rng = np.random.default_rng(seed)
    xs = [_fill(rng, C, N) for N in ns]
    refs = oracle_many(xs, ns, [PARAMS] * len(ns))
    fills = [make_fill(dev(x), N, PARAMS) for x, N in zip(xs, ns)]
    outs = [daq.alloc_out(f) for f in fills]
    for form in ("batch", "again", "noalloc"):
        for o in outs:
            poison_out(o)
        log("%s %s" % (what, form))
        (ctx.daq_process_batch_noalloc if form == "noalloc" else ctx.daq_process_batch)(fills, outs)
        torch.cuda.synchronize()
        for i, (o, r) in enumerate(zip(outs, refs)):
            assert_same(o, r, ctx="%s %s fill %d" % (what, form, i))


@pytest.mark.parametrize("wgs", [1, 2, 4, 7, 8])
@pytest.mark.parametrize("C", [2, 30])
@pytest.mark.parametrize("n", [1, 5, 20])
def test_rounds(wgs, C, n):
    """Tiles of the launch: just under and from eight rounds of the bound on."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    with daq.Context(0) as ctx:
        ctx.set_schedule(512, wgs, 5, 0)
        for tiles in (min(8 * wgs, 16) * cus - 1, min(8 * wgs, 16) * cus):
            each = tiles // n
            ns = [each * TILE - 3] * (n - 1) + [(tiles - each * (n - 1)) * TILE - 300]
            _check(ctx, C, ns, "wgs=%d C=%d n=%d tiles=%d" % (wgs, C, n, tiles))
