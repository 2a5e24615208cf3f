"""daq_gather_islands on tables the library did not write: the packed samples
follow the documented rule (position q holds sample start + q - offset of the
last record with offset <= q), whatever the records' order, lengths and
number. Whole numbers, so equality is exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import dev, log, pad_stride, poison  # noqa: E402


def _table(kind, rng, N):
    """Records (start, stop, offset) whose samples all lie in the fill."""
    if kind == "decreasing":      # neighbouring packed samples come from far apart, down to sample 0
        lens = rng.integers(1, 40, 60)
        starts = np.sort(rng.choice(N - 40, 60, replace=False))[::-1].copy()
        starts[-1] = 0
        starts[0] = N - lens[0]
    elif kind == "single samples":  # more runs than 16-byte words
        starts = np.arange(0, N, 2)
        lens = np.ones(len(starts), np.int64)
    elif kind == "empty records":  # 900 records of no samples inside one segment
        starts = np.concatenate([[5], np.full(900, 7), [N - 700]])
        lens = np.concatenate([[100], np.zeros(900, np.int64), [700]])
    elif kind == "one record":
        starts, lens = np.array([0]), np.array([N])
    else:                          # many: three search steps
        starts = np.arange(0, N - 8, 11)
        lens = rng.integers(1, 9, len(starts))
    offs = np.concatenate([[0], np.cumsum(lens)[:-1]])
    return np.stack([starts, starts + lens, offs], 1).astype(np.int64)


@pytest.mark.parametrize("kind", ["decreasing", "single samples", "empty records", "one record", "many"])
@pytest.mark.parametrize("C,N", [(54, 1000), (1, 4097), (7, 60_001)])
@pytest.mark.parametrize("odd_rows", [False, True])
def test_gather_from_a_table_of_the_callers(kind, C, N, odd_rows):
    rng = np.random.default_rng(C * 7 + N)
    x = pad_stride(rng.integers(-32768, 32768, size=(C, N)).astype(np.int16))
    t = _table(kind, rng, N)
    total = int(t[-1, 2] + t[-1, 1] - t[-1, 0])
    pos = np.arange(total)
    r = np.searchsorted(t[:, 2], pos, side="right") - 1
    want = x[:, t[r, 0] + pos - t[r, 2]]
    stride = daq.padded(total) + (3 if odd_rows else 0)
    out = poison(torch.empty((C, max(stride, 8)), dtype=torch.int16, device="cuda"))
    counts = torch.tensor([len(t), total, 0], dtype=torch.int64, device="cuda")
    fo = daq.FillOut(dev(t), counts, None, out)
    log("gather %s C=%d N=%d odd=%s" % (kind, C, N, odd_rows))
    with daq.Context(0) as ctx:
        ctx.daq_gather_islands(daq.Fill(dev(x), N), fo)
        torch.cuda.synchronize()
    got = out.cpu().numpy()
    np.testing.assert_array_equal(got[:, :total], want)
    assert (got[:, total:] == 0x5A5A).all()
