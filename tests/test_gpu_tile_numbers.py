"""Tiles are numbered over a batch's fills without gaps, their summaries in whole
groups per fill: batches of empty and tiny fills in every place, more fills than
one load of bases covers, fill groups, new and repeated tables, 128 and more
pedestal samples. Whole numbers against the oracle, so equality is exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import assert_same, dev, log, make_fill, oracle_many, pad_stride, poison_out  # noqa: E402

BATCHES = {
    "all empty": [0] * 5,
    "two empty": [0, 0],
    "empty ends": [0, 0, 700, 0, 513, 0, 0],
    "one tile": [0] * 15 + [1],
    "first tile": [512] + [0] * 15,
    "tiles and groups": [511, 512, 513, 16_383, 16_384, 16_385, 0, 20_000],
    "many": None,
}


def _fill(rng, C, N):
    x = rng.integers(995, 1006, size=(C, max(N, 1))).astype(np.int16)
    if N:
        x[0, rng.integers(0, N, N // 200 + 1)] -= 500
    return pad_stride(x)


@pytest.mark.parametrize("what", list(BATCHES))
@pytest.mark.parametrize("C", [3, 40])
@pytest.mark.parametrize("parts", [0, 3])
@pytest.mark.parametrize("ped", [100, 400])
def test_batches(what, C, parts, ped):
    rng = np.random.default_rng(C + ped)
    ns = BATCHES[what] or [int(v) for v in rng.choice([0, 1, 200, 512, 700, 3000, 17_000], size=150)]
    p = {"threshold": -200, "pre": 8, "post": 24, "ped_samples": ped}
    xs = [_fill(rng, C, N) for N in ns]
    refs = oracle_many(xs, ns, [p] * len(ns))
    fills = [make_fill(dev(x), N, p) for x, N in zip(xs, ns)]
    outs = [daq.alloc_out(f) for f in fills]
    with daq.Context(0) as ctx:
        ctx.set_schedule(512, 8, 5, parts)
        for form in ("new", "same", "reversed", "noalloc"):
            order = range(len(ns))[::-1] if form == "reversed" else range(len(ns))
            for o in outs:
                poison_out(o)
            log("%s C=%d parts=%d ped=%d %s" % (what, C, parts, ped, form))
            call = ctx.daq_process_batch_noalloc if form == "noalloc" else ctx.daq_process_batch
            call([fills[i] for i in order], [outs[i] for i in order])
            torch.cuda.synchronize()
            for i, (o, r) in enumerate(zip(outs, refs)):
                assert_same(o, r, ctx="%s fill %d" % (form, i))
