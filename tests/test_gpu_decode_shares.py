"""Decoding launches on both sides of the rule that gives every group of eight
blocks a wave of its own (streams with room for at most 45,056 groups) or shares
the work-groups out by the streams' groups, and compression of a lone fill whose
waves outnumber its groups. Round trips of known rows, exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import log  # noqa: E402
from test_gpu_compress import packed_out, rows  # noqa: E402

GROUP = 512


def _round_trip(xs, Ls, what):
    with daq.Context(0) as ctx:
        outs = [packed_out(x, L) for x, L in zip(xs, Ls)]
        zouts = [daq.alloc_z_out(x.shape[0], o.out.shape[1], device="cuda") for x, o in zip(xs, outs)]
        log(what)
        ctx.daq_compress_batch(outs, zouts)
        backs = [torch.full((x.shape[0], max(daq.padded(L), 8)), -3, dtype=torch.int16, device="cuda")
                 for x, L in zip(xs, Ls)]
        ctx.daq_decompress_batch(zouts, Ls, backs)
        torch.cuda.synchronize()
        for i, (b, o, L) in enumerate(zip(backs, outs, Ls)):
            assert torch.equal(b[:, :L], o.out[:, :L]), "%s fill %d" % (what, i)
            assert bool((b[:, L:] == -3).all())


@pytest.mark.parametrize("C,L", [(11, 4096 * GROUP - 1), (11, 4096 * GROUP), (11, 4096 * GROUP + 1), (1, 1), (1, GROUP),
                                 (54, 4 * GROUP + 1)])
def test_one_stream(C, L):
    _round_trip([rows(C, C, L, "noise")], [L], "C=%d L=%d" % (C, L))


@pytest.mark.parametrize("Ls", [[0, 1, GROUP, 3 * GROUP + 7], [176 * GROUP] * 16, [177 * GROUP] * 16,
                                [176 * GROUP] + [5] * 15, [40 * GROUP] + [0] * 16, [400 * GROUP] + [7] * 16])
def test_streams_of_one_launch_and_more(Ls):
    _round_trip([rows(i, 16, L, ["noise", "wide"][i % 2]) for i, L in enumerate(Ls)], Ls, "streams %s" % Ls[:2])
