"""Fills of few channels, on both sides of the rules that give each tile of the
split schedule's scan one wave or four: up to 28 channels, and launches of at
least two tiles of 512 samples per CU. Pedestals within the scan and from a
kernel of their own, every entry form, fills of several lengths in one launch.
Whole numbers against the oracle, so equality is exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import assert_same, dev, log, make_fill, oracle_many, oracle_result, pad_stride, poison_out, run  # noqa: E402

TILE = 512


def _fill(rng, C, N):
    """Any int16 in the first samples, then noise with crossings at tile edges
    and between, in the last channel as well as the first."""
    x = rng.integers(995, 1006, size=(C, N)).astype(np.int16)
    at = np.unique(np.concatenate([rng.integers(0, N, N // 700 + 2), np.arange(0, N, 41 * TILE), [N - 1]]))
    x[0, at[::2]] -= 500
    x[C - 1, at[1::2]] -= 500
    k = min(N, 60)
    x[:, :k] = rng.integers(900, 1100, size=(C, k))
    return pad_stride(x)


def _params(np_=100):
    return {"threshold": -220, "pre": 8, "post": 24, "ped_samples": np_}


@pytest.mark.parametrize("C", [1, 2, 6, 7, 8, 14, 15, 17, 28, 29])
@pytest.mark.parametrize("tiles", [511, 512, 1100])
def test_one_fill(C, tiles):
    rng = np.random.default_rng(C * 7 + tiles)
    with daq.Context(0) as ctx:
        for N in (tiles * TILE, tiles * TILE - 509):
            x = _fill(rng, C, N)
            for np_ in (100, 1, 128, 129):
                ref = oracle_result(x, N, _params(np_))
                f = make_fill(dev(x), N, _params(np_))
                for mode in ("chop", "batch"):
                    log("C=%d N=%d np=%d %s" % (C, N, np_, mode))
                    o = daq.alloc_out(f)
                    run(ctx, mode, [f], [o])
                    assert_same(o, ref, ctx="np=%d %s" % (np_, mode))


@pytest.mark.parametrize("C", [3, 12, 28, 29])
@pytest.mark.parametrize("n", [2, 5, 16, 17, 30])
@pytest.mark.parametrize("parts", [0, 2])
def test_batches_of_uneven_fills(C, n, parts):
    rng = np.random.default_rng(C * 100 + n)
    ns = [int(v) for v in rng.choice([0, 1, 7, 511, 512, 513, 16_384, 16_385, 40_001, 90_000], size=n)]
    ns[n // 2] = 300_007
    xs = [_fill(rng, C if i % 3 else max(1, C - 2), N) if N else pad_stride(np.zeros((C, 8), np.int16))
          for i, N in enumerate(ns)]
    for np_ in (100, 500):
        ps = [_params(np_)] * n
        refs = oracle_many(xs, ns, ps)
        fills = [make_fill(dev(x), N, p) for x, N, p in zip(xs, ns, ps)]
        with daq.Context(0) as ctx:
            ctx.set_schedule(512, 8, 5, parts)
            for form in ("new", "same", "noalloc"):
                outs = [poison_out(daq.alloc_out(f)) for f in fills] if form == "new" else outs  # noqa: F821
                for o in outs:
                    poison_out(o)
                log("C=%d n=%d parts=%d np=%d %s" % (C, n, parts, np_, form))
                if form == "noalloc":
                    ctx.daq_process_batch_noalloc(fills, outs)
                else:
                    ctx.daq_process_batch(fills, outs)
                torch.cuda.synchronize()
                for i, (o, r) in enumerate(zip(outs, refs)):
                    assert_same(o, r, ctx="%s fill %d" % (form, i))
