"""The tuner times no two schedules that launch the same kernels: of the split
variant's, which depend on the number of fill groups alone, one for each number,
all with the work-groups that a new context has (the Q-method's pass takes them,
and the tuner does not time it). In a child process, since the library reads
DAQ_LOG once per process."""
import os
import re
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU machines
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import log  # noqa: E402

TESTS = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(TESTS)

CHILD = r"""
import torch
import paper_1611_04959_amd as daq
fills = [daq.Fill(torch.full((54, 20_000), 1800, dtype=torch.int16, device="cuda"), 20_000) for _ in range(8)]
outs = [daq.alloc_out(f) for f in fills]
with daq.Context(0) as ctx:
    s = ctx.get_schedule()
    print("default", s.threads, s.wgs_per_cu, flush=True)
    ctx.daq_autotune(fills, outs)
"""


def test_one_candidate_for_each_number_of_fill_groups():
    env = {k: v for k, v in os.environ.items() if not k.startswith("DAQ_")}
    env.update(DAQ_LOG="2", PYTHONPATH=os.pathsep.join([ROOT, TESTS]))
    log("tuner in a child process")
    r = subprocess.run([sys.executable, "-c", CHILD], capture_output=True, text=True, env=env, timeout=100)
    assert r.returncode == 0, r.stderr
    default = [int(v) for v in re.search(r"default (\d+) (\d+)", r.stdout).groups()]
    timed = [tuple(int(v) for v in m) for m in re.findall(r"autotune: schedule (\d+)/(\d+)/(\d+)/(\d+) median", r.stderr)]
    assert len(timed) == len(set(timed)) >= 10, timed
    split = [t for t in timed if t[2] == 5]
    assert sorted(t[3] for t in split) == [0, 2, 3, 4], split
    assert all(list(t[:2]) == default for t in split), split
