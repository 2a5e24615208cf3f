"""Batches on both sides of the sizes that take one kernel after the scan: up to
four fills of 2^20 samples together. Against the oracle, exactly."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

import paper_1611_04959_amd as daq  # noqa: E402
from test_gpu_bounded_scan import _check  # noqa: E402


@pytest.mark.parametrize("n", [2, 4, 5])
def test_sizes_around_the_emit_pass(n):
    with daq.Context(0) as ctx:
        for samples in (1 << 20, (1 << 20) + 1):
            each = samples // n
            ns = [each] * (n - 1) + [samples - each * (n - 1)]
            _check(ctx, 3, ns, "n=%d samples=%d" % (n, samples))
