"""daq_process_batch_noalloc close to its scratch limit: as many tiny or empty
fills as fit, and a few very long ones. The tile summaries lie behind the
documented bytes and must fit too, whatever the fills. Exact, against the
oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import assert_same, dev, log, make_fill, oracle_many, pad_stride, poison_out  # noqa: E402


@pytest.mark.parametrize("kind", ["empty", "one sample", "mixed"])
def test_as_many_tiny_fills_as_fit(kind):
    """Every fill reads the same raw row of 8 samples (or none); each has a
    record, counts and a packed row of its own."""
    raw = torch.tensor([[1000, 1000, 1000, 1000, 500, 1000, 1000, 1000]], dtype=torch.int16, device="cuda")
    most = 170_000
    length = {"empty": [0], "one sample": [1], "mixed": [8, 0, 1, 5]}[kind]
    lib = daq.load_library()

    def array(n):
        fa = (daq.daq_fill * n)()
        for i in range(n):
            fa[i] = daq.daq_fill(raw.data_ptr(), length[i % len(length)], 8, 1, 1, -100, 0, 0, 0)
        return fa

    fa = array(most)
    lo, hi = 1, most  # the largest batch that fits
    while lo < hi:
        mid = (lo + hi + 1) // 2
        if lib.daq_noalloc_scratch_bytes(fa, mid) <= daq.DAQ_NOALLOC_SCRATCH_BYTES:
            lo = mid
        else:
            hi = mid - 1
    n = lo
    assert 1000 < n < most
    isl = torch.full((n, 3), -1, dtype=torch.int64, device="cuda")
    counts = torch.full((n, 3), -1, dtype=torch.int64, device="cuda")
    ped = torch.full((n, 1), -1, dtype=torch.int32, device="cuda")
    out = torch.full((n, 8), 77, dtype=torch.int16, device="cuda")
    oa = (daq.daq_fill_out * n)()
    for i in range(n):
        oa[i] = daq.daq_fill_out(isl.data_ptr() + 24 * i, 1, counts.data_ptr() + 24 * i, ped.data_ptr() + 4 * i,
                                 out.data_ptr() + 16 * i, 8)
    log("%s: %d fills" % (kind, n))
    with daq.Context(0) as ctx:
        assert lib.daq_process_batch_noalloc(ctx.handle, fa, oa, n, None) == daq.DAQ_OK
        torch.cuda.synchronize()
        more = (daq.daq_fill_out * most)(*([oa[0]] * most))
        assert lib.daq_process_batch_noalloc(ctx.handle, fa, more, most, None) == daq.DAQ_ERANGE
    ls = np.array([length[i % len(length)] for i in range(n)])
    found = (ls > 4).astype(np.int64)  # the crossing is sample 4
    np.testing.assert_array_equal(counts.cpu().numpy(), np.stack([found, found, 0 * found], 1))
    np.testing.assert_array_equal(ped.cpu().numpy()[:, 0], np.where(ls > 0, 1000, 0))
    got = isl.cpu().numpy()
    assert (got[found == 1] == [4, 5, 0]).all() and (got[found == 0] == -1).all()
    rows = out.cpu().numpy()
    assert (rows[found == 1, 0] == 500).all() and (rows[:, 1:] == 77).all() and (rows[found == 0, 0] == 77).all()


def test_long_fills():
    rng = np.random.default_rng(4)
    p = {"threshold": -200, "pre": 8, "post": 24, "ped_samples": 100}
    ns = [25_000_003, 20_000_000, 16_777_217, 9_999_999]
    xs = []
    for N in ns:
        x = rng.integers(995, 1006, size=(1, N)).astype(np.int16)
        x[0, rng.integers(0, N, N // 3000)] -= 500
        xs.append(pad_stride(x))
    refs = oracle_many(xs, ns, [p] * len(ns))
    fills = [make_fill(dev(x), N, p) for x, N in zip(xs, ns)]
    need = daq.noalloc_scratch_bytes(fills)
    assert daq.DAQ_NOALLOC_SCRATCH_BYTES * 0.7 < need <= daq.DAQ_NOALLOC_SCRATCH_BYTES, need
    outs = [poison_out(daq.alloc_out(f)) for f in fills]
    log("long fills, %d scratch bytes" % need)
    with daq.Context(0) as ctx:
        for call in (ctx.daq_process_batch_noalloc, ctx.daq_process_batch):
            for o in outs:
                poison_out(o)
            call(fills, outs)
            torch.cuda.synchronize()
            for i, (o, r) in enumerate(zip(outs, refs)):
                assert_same(o, r, ctx="fill %d" % i)
