"""Pedestals around the length (512 samples) from which a kernel with a work-group
per channel computes them, alone and beside shorter ones in a launch, over any
int16 samples: every entry form against the oracle, exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import assert_same, dev, log, make_fill, oracle_many, pad_stride, poison_out, run  # noqa: E402

LENGTHS = [511, 512, 513, 519, 2048, 16_383, 16_385, 50_000]


def _fill(rng, C, N, np_):
    x = pad_stride(rng.integers(-32768, 32768, size=(C, N)).astype(np.int16))
    S = x[:, :N].astype(np.int64).sum(0)
    return x, {"threshold": int(np.quantile(S, 0.03)), "pre": 3, "post": 9, "ped_samples": np_}


@pytest.mark.parametrize("C", [1, 5, 54, 70])
def test_one_fill(C):
    rng = np.random.default_rng(C)
    with daq.Context(0) as ctx:
        for np_ in LENGTHS:
            x, p = _fill(rng, C, 30_011, np_)
            ref = oracle_many([x], [30_011], [p])[0]
            f = make_fill(dev(x), 30_011, p)
            for mode in ("chop", "twopass", "batch"):
                log("C=%d np=%d %s" % (C, np_, mode))
                o = daq.alloc_out(f)
                run(ctx, mode, [f], [o])
                assert_same(o, ref, ctx="np=%d %s" % (np_, mode))


@pytest.mark.parametrize("n", [2, 6, 20])
def test_long_and_short_ones_in_one_launch(n):
    rng = np.random.default_rng(n)
    cs = [int(c) for c in rng.choice([1, 3, 54, 70], size=n)]
    ns = [int(v) for v in rng.choice([1, 100, 513, 9000, 30_011], size=n)]
    ns[0] = 30_011
    cases = [_fill(rng, C, N, int(rng.choice([1, 100, 129, 400] + LENGTHS))) for C, N in zip(cs, ns)]
    cases[0][1]["ped_samples"] = 5000
    xs, ps = [c[0] for c in cases], [c[1] for c in cases]
    refs = oracle_many(xs, ns, ps)
    fills = [make_fill(dev(x), N, p) for x, N, p in zip(xs, ns, ps)]
    outs = [daq.alloc_out(f) for f in fills]
    with daq.Context(0) as ctx:
        for form in ("batch", "again", "noalloc", "both", "groups"):
            for o in outs:
                poison_out(o)
            log("n=%d %s" % (n, form))
            if form == "both":
                qs = [daq.alloc_q_out(f, acc=False) for f in fills]
                for q in qs:
                    q.ped = None
                lib = daq.load_library()
                fa = (daq.daq_fill * n)(*[f.c_struct() for f in fills])
                oa = (daq.daq_fill_out * n)(*[o.c_struct() for o in outs])
                qa = (daq.daq_q_out * n)(*[q.c_struct() for q in qs])
                assert lib.daq_process_batch_q(ctx.handle, fa, oa, qa, n, None) == daq.DAQ_OK
            elif form == "noalloc":
                ctx.daq_process_batch_noalloc(fills, outs)
            else:
                if form == "groups":
                    ctx.set_schedule(512, 8, 5, 2)
                ctx.daq_process_batch(fills, outs)
            torch.cuda.synchronize()
            for i, (o, r) in enumerate(zip(outs, refs)):
                assert_same(o, r, ctx="%s fill %d" % (form, i))
            if form == "both":
                for i, (q, x, N, p) in enumerate(zip(qs, xs, ns, ps)):
                    ref = oracle.qmethod(x, N, ped_samples=p["ped_samples"])[1]
                    np.testing.assert_array_equal(q.qsum.cpu().numpy()[:len(ref)], ref, err_msg="qsum %d" % i)
