"""Compression of a lone fill whose launch has more waves than the fill has
groups of eight blocks, since its rows have room for many more samples than
they hold: most waves have no group, and the last one that has writes the
stream's length. Against the oracle, exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_04959_amd as daq  # noqa: E402
from gpu_util import log  # noqa: E402
from test_gpu_compress import check, packed_out, rows  # noqa: E402


@pytest.mark.parametrize("C,L,room", [(54, 20_000, 180_000), (54, 512, 180_000), (54, 180_000, 180_000),
                                      (3, 100, 4_000_000), (54, 0, 180_000), (1, 64, 64)])
def test_a_lone_fill_with_more_waves_than_groups(C, L, room):
    x = np.concatenate([rows(1, C, L, "noise")[:, :L], np.zeros((C, room - L), np.int16)], 1)
    o = packed_out(x, L)
    z = daq.alloc_z_out(C, o.out.shape[1], device="cuda")
    log("C=%d L=%d room %d" % (C, L, room))
    with daq.Context(0) as ctx:
        ctx.daq_compress_batch([o], [z])
        torch.cuda.synchronize()
    check(z, x, L, "lone")
