"""The compression kernels where their paths part: every block width (16-bit
halves up to 16 bits, one 64-bit value up to 8, two up to 16, the general path
at 17), samples near the limits of the two-at-a-time codes, whole groups of
eight blocks and ragged ends, and batches whose fills are so uneven that the
launch's work-groups are shared out very unequally. Exact, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import log  # noqa: E402
from test_gpu_compress import check, packed_out, rows  # noqa: E402


def _round_trip(xs, Ls, what):
    with daq.Context(0) as ctx:
        outs = [packed_out(x, L) for x, L in zip(xs, Ls)]
        zouts = [daq.alloc_z_out(x.shape[0], o.out.shape[1], device="cuda") for x, o in zip(xs, outs)]
        log("compress " + what)
        ctx.daq_compress_batch(outs, zouts)
        torch.cuda.synchronize()
        for i, (z, x, L) in enumerate(zip(zouts, xs, Ls)):
            check(z, x, L, "%s fill %d" % (what, i))
        backs = [torch.full((x.shape[0], max(daq.padded(L), 8)), -3, dtype=torch.int16, device="cuda")
                 for x, L in zip(xs, Ls)]
        log("decompress " + what)
        ctx.daq_decompress_batch(zouts, Ls, backs)
        torch.cuda.synchronize()
        for i, (b, x, L) in enumerate(zip(backs, xs, Ls)):
            got = b.cpu().numpy()
            np.testing.assert_array_equal(got[:, :L], x[:, :L], err_msg="%s fill %d" % (what, i))
            assert (got[:, L:] == -3).all()


@pytest.mark.parametrize("w", list(range(18)))
def test_every_width(w):
    """Blocks whose largest code has exactly w bits, beside blocks of any width
    up to w, at sample levels where two-at-a-time differences do and do not
    fit."""
    rng = np.random.default_rng(w)
    big = [0] if w == 0 else [(1 << (w - 1)) // 2, -((1 << (w - 1)) // 2) - ((1 << (w - 1)) & 1)]
    xs, Ls = [], []
    for L in (512, 64 * 24, 64 * 24 + 17):
        x = np.zeros((5, L), np.int64)
        for c, level in enumerate((0, 16383, -16384, 1800, 32767)):
            step = np.zeros(L, np.int64)
            for k in range(0, L, 64):
                m = w if (k // 64) % 3 else int(rng.integers(0, w + 1))
                half = (1 << m) // 4
                d = rng.integers(-half, half + 1, size=min(64, L - k))
                if m == w and len(d) > 5:
                    d[5] = big[int(rng.integers(0, len(big)))]
                step[k:k + len(d)] = d
            v = level
            for t in range(L):  # a walk that stays in int16: turn back at the limits
                d = step[t]
                if not -32768 <= v + d <= 32767:
                    d = -d if -32768 <= v - d <= 32767 else 0
                v += d
                x[c, t] = v
        if w == 17:
            x[0, ::2], x[0, 1::2] = -32768, 32767
        xs.append(x.astype(np.int16))
        Ls.append(L)
    _round_trip(xs, Ls, "width %d" % w)


@pytest.mark.parametrize("n", [2, 15, 16, 17])
def test_uneven_fills_share_a_launch(n):
    rng = np.random.default_rng(n)
    Ls = [int(v) for v in rng.choice([0, 1, 63, 64, 511, 512, 513, 3000], size=n)]
    Ls[n // 2] = 60_997
    xs = [rows(i, 54 if L > 5000 else 1 + i % 7, L, ["noise", "mixed"][i % 2]) for i, L in enumerate(Ls)]
    _round_trip(xs, Ls, "uneven %d" % n)


def test_empty_fills_only():
    _round_trip([rows(i, 3, 0, "flat") for i in range(3)], [0, 0, 0], "empty")
