"""daq_gather_islands on tables that do not begin at packed position 0 (the tail
of an island table): positions before the first record continue it to the left,
as start + q - offset says. And on records that leave the fill: a sample outside
the n_channels * row_stride elements of the fill is not read and becomes 0.
Whole numbers, so equality is exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import dev, log, pad_stride, poison  # noqa: E402

RECORDS = 40


def _check(t, C, N, odd_rows, what):
    """t: records whose offsets follow each other, the first one's at any place."""
    rng = np.random.default_rng(C + N)
    x = pad_stride(rng.integers(-32768, 32768, size=(C, N)).astype(np.int16))
    total = int(t[-1, 2] + t[-1, 1] - t[-1, 0])
    pos = np.arange(total)
    r = np.maximum(np.searchsorted(t[:, 2], pos, side="right") - 1, 0)
    at = np.arange(C)[:, None] * x.shape[1] + (t[r, 0] + pos - t[r, 2])[None, :]
    inside = (at >= 0) & (at < x.size)
    want = np.where(inside, x.reshape(-1)[np.where(inside, at, 0)], 0).astype(np.int16)
    out = poison(torch.empty((C, daq.padded(total) + (3 if odd_rows else 8)), dtype=torch.int16, device="cuda"))
    counts = torch.tensor([len(t), total, 0], dtype=torch.int64, device="cuda")
    log("%s C=%d N=%d odd=%s" % (what, C, N, odd_rows))
    with daq.Context(0) as ctx:
        ctx.daq_gather_islands(daq.Fill(dev(x), N), daq.FillOut(dev(t), counts, None, out))
        torch.cuda.synchronize()
    got = out.cpu().numpy()
    np.testing.assert_array_equal(got[:, :total], want)
    assert (got[:, total:] == 0x5A5A).all()


def _records(rng, starts, first):
    lens = rng.integers(1, 40, len(starts))
    offs = first + np.concatenate([[0], np.cumsum(lens)[:-1]])
    return np.stack([starts, starts + lens, offs], 1).astype(np.int64)


@pytest.mark.parametrize("first", [1, 5, 8, 9, 511, 512, 700, 1030])
@pytest.mark.parametrize("C,N", [(1, 4097), (54, 5003)])
@pytest.mark.parametrize("odd_rows", [False, True])
def test_a_table_that_begins_after_position_0(first, C, N, odd_rows):
    rng = np.random.default_rng(first)
    starts = np.sort(rng.choice(np.arange(1100, N - 40), RECORDS, replace=False))
    _check(_records(rng, starts, first), C, N, odd_rows, "first offset %d" % first)


@pytest.mark.parametrize("C,N", [(1, 4097), (5, 5003)])
@pytest.mark.parametrize("odd_rows", [False, True])
def test_records_that_leave_the_fill(C, N, odd_rows):
    rng = np.random.default_rng(C)
    starts = rng.integers(0, N - 40, RECORDS)
    starts[::4] = [-7, -30_000, N - 3, N + 9, 2_000_000_000, -2_000_000_000, -1, N - 8, 6 * N, -5 * N]
    for first in (0, 3):
        _check(_records(rng, starts, first), C, N, odd_rows, "outside, first offset %d" % first)
    # more records than one segment's table holds: empty ones before the last
    t = _records(rng, starts, 0)
    empty = np.repeat([[7, 7, t[-1, 2]]], 600, 0)
    _check(np.concatenate([t[:-1], empty, t[-1:]]).astype(np.int64), C, N, odd_rows, "outside, empty records")
