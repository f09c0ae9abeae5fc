"""The in-kernel clock stamps (libecspmv_trace.so, the library's sources built with -DECS_TRACE) and the script that
reads them: a short run on the small config, in a process of its own because it loads the stamped library in place of
the product one.  The stamped kernel must still compute y (the script's launches are checked against the oracle's band
by the parity tests of the product library; here the order of the stamped points is what is checked)."""
import json
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2507_12205_amd import timeline

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def assert_in_order(by):
    """Every wavefront passes every point after it started, in the launches that stamped the point.  From one point to another launches
    differ, so only points that lie hundreds of nanoseconds apart are compared: header here, first barrier, second barrier."""
    for k, row in by.items():
        if k:
            assert row["before_own_start"] == 0 and row["own_start_median_us"] <= row["median_us"], row
    med = [by[k]["median_us"] for k in (23, 1, 4, 12)]
    assert all(a <= b for a, b in zip(med, med[1:])), med


@pytest.mark.gpu
def test_timeline_runs_and_points_come_in_order(tmp_path):
    from paper_2507_12205_amd import build as B
    if not os.path.exists(B.TRACE_LIB):
        pytest.fail(f"{B.TRACE_LIB} is missing: __graft_entry__.build() makes it")
    out = tmp_path / "t.json"
    env = dict(os.environ)
    env.pop("ECSPMV_LIB", None)
    r = subprocess.run([sys.executable, "-m", "paper_2507_12205_amd.timeline", "--config", "0", "--shape", "0",
                        "--copies", "2", "--launches", "6", "--json", str(out)],
                       cwd=ROOT, env=env, capture_output=True, text=True, timeout=240)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    d = json.loads(out.read_text())
    by = {row["stamp"]: row for row in d["stamps"]}
    for k in (0, 1, 2, 3, 4, 12):
        assert k in by, f"stamp {k} missing"
    assert_in_order(by)
    assert 0.0 < d["kernel_span_us"] < 100.0 and d["us_per_launch_stamps_off"] > 0.0
    assert 500.0 < d["stamp_clock_mhz"] < 3000.0


@pytest.mark.gpu
def test_points_where_x_comes_first(tmp_path):
    """A wide x and no block sets: the first chunks are requested once this wavefront's pieces are in LDS (times from the start of the
    wavefronts that passed a point, in the launches that stamped it).  Between the header and that point lie the stores of 16 wavefronts
    x 2 KB, 0.11 us of an LDS that takes 128 bytes a cycle at 2.3 GHz, half of it for the median wavefront; where nothing lies
    between two points they are 0.01-0.02 us apart."""
    out = tmp_path / "t.json"
    r = subprocess.run([sys.executable, "-m", "paper_2507_12205_amd.timeline", "--config", "2", "--shape", "1", "--delta-bits", "8",
                        "--max-granularity", "1", "--copies", "2", "--launches", "8", "--json", str(out)],
                       cwd=ROOT, env={k: v for k, v in os.environ.items() if k != "ECSPMV_LIB"}, capture_output=True, text=True, timeout=240)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    by = {row["stamp"]: row for row in json.loads(out.read_text())["stamps"]}
    assert_in_order(by)
    after = {k: by[k]["median_us"] - by[k]["own_start_median_us"] for k in (1, 2, 4)}
    assert after[2] > after[1] + 0.05 and after[4] > after[2], after


def stamps(starts, passed):
    """a launch of one workgroup per entry: clock at the start, at the point and at the end, constant-rate clock at start and end"""
    T = np.zeros((2, len(starts), 1, 8), dtype=np.int64)
    for i, s in enumerate(starts):
        clock, real = 10 ** 9 + 7 * i, 5000 + s                        # 2000 MHz and 100 MHz
        T[:, i, 0, :5] = clock, clock + passed, clock + 4000, real, real + 200
    return T


def test_order_does_not_depend_on_when_launches_start():
    """a launch whose wavefronts start sooner than those of the launch the start was taken from: every wavefront is in order, the medians
    of two launches are not; and a wavefront that passes a point before it started is found"""
    early, late, by = [0, 10, 20], [0, 23, 40], {}
    for k, starts, passed in ((22, late, 4), (23, early, 6), (1, late, 600), (4, early, 1500), (12, late, 3000)):
        for row in timeline.rows_of(k, str(k), stamps(starts, passed), 2000.0, first=not by):
            by[row["stamp"]] = row
    assert by[0]["median_us"] > by[23]["median_us"]
    assert_in_order(by)
    [row] = timeline.rows_of(23, "23", stamps(early, -1), 2000.0, first=False)
    with pytest.raises(AssertionError):
        assert_in_order({**by, 23: row})
