"""The benchmark's roofline on the CPU: a share of the peak is one of bytes that were moved."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


def test_roofline_counts_the_bytes_moved():
    """8192 x 4096 in binary32, 20 steps at 0.229 ms: six launches of three steps by their
    counters and two single steps."""
    rec = {"hbm_bytes_per_launch": 2924276422, "steps_per_launch": 3}
    single = 33468220 * 72
    r = bench.step_roofline(rec, single, 20, 0.22937e-3)
    moved = (6 * 2924276422 + 2 * single) / 20
    assert r["traffic"] == pytest.approx(moved, rel=1e-9)
    assert r["achieved"] == pytest.approx(moved / 0.22937e-3 / 1e9, rel=1e-4)
    assert r["frac"] == pytest.approx(r["achieved"] / bench.HBM_PEAK_GBS, abs=1e-4) and r["frac"] < 1
    assert r["single_step_gbs"] > bench.HBM_PEAK_GBS


def test_roofline_without_counters_gives_no_share():
    r = bench.step_roofline(None, 33468220 * 72, 20, 0.22937e-3)
    assert r["frac"] is None and r["achieved"] is None and r["traffic"] is None


def test_roofline_of_single_steps():
    r = bench.step_roofline({"hbm_bytes_per_launch": 2.5e9}, 2.4e9, 7, 0.5e-3)
    assert r["frac"] == pytest.approx(2.5e9 / 0.5e-3 / 1e9 / bench.HBM_PEAK_GBS, abs=1e-4)
