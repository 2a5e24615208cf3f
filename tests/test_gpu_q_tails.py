"""Fills whose last group of 8 samples is not whole, through the Q-method and
both methods on one read, in launches on both sides of the rule that loads
accumulator rows together or one by one (96 MiB of raw samples). The accumulator
rows hold the fill's samples rounded up to a multiple of 4 and no more; what lies
past a fill's samples, or past its last row, stays as it was. Exact, against the
oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import oracle  # noqa: E402
import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import assert_same, dev, log, make_fill, oracle_result, pad_stride, poison_out  # noqa: E402

PARAMS = {"threshold": -200, "pre": 8, "post": 24, "ped_samples": 100}
GUARD = 64


def _case(rng, C, N):
    x = rng.integers(995, 1006, size=(C, N)).astype(np.int16)
    x[0, rng.integers(0, N, N // 300 + 1)] -= 500
    x = pad_stride(x)
    stride = (N + 3) // 4 * 4
    acc = rng.integers(-2 ** 31, 2 ** 31, size=C * stride + GUARD, dtype=np.int64).astype(np.int32)
    want = acc.copy()
    view = want[:C * stride].reshape(C, stride)
    sums = np.zeros((C, N), np.int32)
    _, qsum = oracle.qmethod(x, N, acc=sums)
    view[:, :N] = (view[:, :N].view(np.uint32) + sums.view(np.uint32)).view(np.int32)
    return x, stride, acc, want, qsum


def _run(C, ns, threads, what):
    rng = np.random.default_rng(sum(ns) + C)
    cases = [_case(rng, C, N) for N in ns]
    fills = [make_fill(dev(x), N, PARAMS) for (x, *_), N in zip(cases, ns)]
    with daq.Context(0) as ctx:
        ctx.set_schedule(threads, 8, 5, 0)
        lib = daq.load_library()
        for both in (False, True):
            log("%s threads=%d both=%s" % (what, threads, both))
            accs = [dev(c[2]) for c in cases]
            qs = [torch.full((len(c[4]),), -9, dtype=torch.int64, device="cuda") for c in cases]
            n = len(ns)
            fa = (daq.daq_fill * n)(*[f.c_struct() for f in fills])
            qa = (daq.daq_q_out * n)(*[daq.daq_q_out(q.data_ptr(), a.data_ptr(), c[1], None)
                                       for q, a, c in zip(qs, accs, cases)])
            if both:
                outs = [poison_out(daq.alloc_out(f)) for f in fills]
                oa = (daq.daq_fill_out * n)(*[o.c_struct() for o in outs])
                assert lib.daq_process_batch_q(ctx.handle, fa, oa, qa, n, None) == daq.DAQ_OK
            else:
                assert lib.daq_qmethod_batch(ctx.handle, fa, qa, n, None) == daq.DAQ_OK
            torch.cuda.synchronize()
            for i, (c, a, q, N) in enumerate(zip(cases, accs, qs, ns)):
                np.testing.assert_array_equal(a.cpu().numpy(), c[3], err_msg="%s acc %d" % (what, i))
                np.testing.assert_array_equal(q.cpu().numpy(), c[4], err_msg="%s qsum %d" % (what, i))
                if both:
                    assert_same(outs[i], oracle_result(c[0], N, PARAMS), ctx="%s fill %d" % (what, i))


@pytest.mark.parametrize("threads", [256, 512])
@pytest.mark.parametrize("tail", range(8))
def test_small_launches(tail, threads):
    for C in (1, 4, 5, 54):
        _run(C, [tail + 1, 2048 + tail, 4096 + tail, 20_000 + tail], threads, "tail=%d C=%d" % (tail, C))


@pytest.mark.parametrize("tail", [0, 1, 3, 4, 5, 7])
def test_large_launches(tail):
    _run(28, [610_000 + tail] * 3 + [5000 + tail], 512, "large tail=%d" % tail)
