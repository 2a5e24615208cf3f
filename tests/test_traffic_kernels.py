"""traffic.py knows the chop's kernels: all that the library's sources hold, and
which of them opens a launch. On synthetic rocprofv3 CSV files."""
import csv
import os
import re

from paper_1611_04959_amd import traffic
from test_traffic_tool import TRACE_FIELDS, write_counters

CSRC = os.path.join(os.path.dirname(traffic.__file__), "csrc")
# kernels of chop_kernels.hip that are no part of a chop launch
OTHERS = {"k_q_pass", "k_unpack12", "k_gather"}


def _full(name):
    return "void daqk::(anonymous namespace)::%s(daqk::KArgs)" % name


def test_every_chop_kernel_is_counted():
    with open(os.path.join(CSRC, "chop_kernels.hip")) as fh:
        names = set(re.findall(r"__global__[^;{]*?\b(k_\w+)\(", fh.read()))
    assert names - OTHERS == set(traffic.PASS_KERNELS)
    assert set(traffic.OPEN_KERNELS) <= set(traffic.PASS_KERNELS)


def test_a_batch_that_is_new_each_time_is_counted_with_its_scan(tmp_path):
    """Launches that open with k_scan_put; and a run whose first launch alone does."""
    write_counters(tmp_path / "cf", "FETCH_SIZE", [(1, "copyBuffer", 64 * 1024)])
    write_counters(tmp_path / "cw", "WRITE_SIZE", [(1, "copyBuffer", 64 * 1024)])
    for put, scan in ((3, 0), (1, 4)):
        d = tmp_path / ("%d_%d" % (put, scan))
        names = [_full("k_scan_put<true, false>")] * put + [_full("k_scan_pass<true, true, false>")] * scan
        rows = [(10 * i, n, 100.0 if "put" in n else 90.0) for i, n in enumerate(names)]
        rows += [(10 * i + 1, _full("k_edge_pass"), 7.0) for i in range(len(names))]
        write_counters(d / "f", "FETCH_SIZE", rows)
        write_counters(d / "w", "WRITE_SIZE", [(n, name, 1.0) for n, name, _ in rows])
        res = traffic.summarize(str(d / "f"), str(d / "w"), str(tmp_path / "cf"), str(tmp_path / "cw"),
                                str(tmp_path / "t.json"), mib=64)
        kept = "k_scan_put" if put > scan else "k_scan_pass"
        assert set(res["kernels"]) == {kept, "k_edge_pass"}
        assert res["bytes_per_launch"] == round(((100.0 if put > scan else 90.0) + 7.0 + 2.0) * 1024)


def test_launches_that_open_with_either_scan(tmp_path, capsys):
    path = tmp_path / "trace.csv"
    t, rows = 1000, []
    for i in range(4):
        for name, d in (("k_scan_put<false, false>" if i % 2 else "k_scan_pass<true, false, false>", 20), ("k_emit_pass", 10)):
            rows.append((_full(name), t * 1000, (t + d) * 1000, "0"))
            t += d
    with open(path, "w", newline="") as fh:
        w = csv.writer(fh)
        w.writerow(TRACE_FIELDS + ["Stream_Id"])
        w.writerows(rows)
    traffic.tail(str(path), 4)
    assert "last 4 launches (first kernel start to last kernel end): 30.0 us" in capsys.readouterr().out
    assert traffic.streams(str(path), 4)["streams"] == {"0": 4}
