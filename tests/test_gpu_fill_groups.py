"""Batches cut into fill groups, each on a stream of its own, with fills longer
than one segment of 589,824 samples: a group's segment summaries are made of
its own fills' tile summaries and of nobody else's. Whole numbers against the
oracle, so equality is exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import assert_same, dev, log, make_fill, oracle_many, pad_stride, poison_out  # noqa: E402

SEGMENT = 512 * 1152
LENGTHS = [SEGMENT + 1, 2 * SEGMENT + 12_345, 5000, SEGMENT + 16_387]
WINDOWS = [(0, 0), (8, 24), (40, 700)]


def _fill(rng, N):
    """Two channels of noise with crossings at the segments' edges and between."""
    x = rng.integers(995, 1006, size=(2, N)).astype(np.int16)
    at = np.concatenate([rng.integers(0, N, N // 500), [0, N - 1, SEGMENT - 1, SEGMENT, SEGMENT + 40, 2 * SEGMENT]])
    x[0, at[at < N]] -= 500
    return pad_stride(x)


@pytest.mark.parametrize("parts", [2, 3, 4])
@pytest.mark.parametrize("n", [4, 7])
def test_segments_of_long_fills_in_every_fill_group(parts, n):
    """Two batches of other fills in one context, so that summaries left from
    the first are wrong for the second."""
    rng = np.random.default_rng(10 * parts + n)
    with daq.Context(0) as ctx:
        ctx.set_schedule(512, 8, 5, parts)
        for batch in range(2):
            ns = [LENGTHS[(i + batch) % 4] for i in range(n)]
            ps = [dict(zip(("pre", "post"), WINDOWS[i % 3]), threshold=-200, ped_samples=100) for i in range(n)]
            xs = [_fill(rng, N) for N in ns]
            refs = oracle_many(xs, ns, ps)
            fills = [make_fill(dev(x), N, p) for x, N, p in zip(xs, ns, ps)]
            outs = [poison_out(daq.alloc_out(f)) for f in fills]
            log("parts=%d n=%d batch %d" % (parts, n, batch))
            ctx.daq_process_batch(fills, outs)
            torch.cuda.synchronize()
            for i, (o, r) in enumerate(zip(outs, refs)):
                assert_same(o, r, ctx="batch %d fill %d" % (batch, i))
