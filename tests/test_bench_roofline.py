"""The benchmark's roofline figures are those of the launches that it timed: the
committed counters hold one window (the middle of the whole run), so bytes,
flops and instructions go by the units of work of the timed launches, not by
those of the recorded ones (a short run clips a third of the recorded window's
pairs and would print an issue rate above the peak)."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("share", [1.0, 0.25])
def test_counters_scale_with_the_units(monkeypatch, share):
    sys.path.insert(0, ROOT)
    import bench
    records = {"traffic-json": {"bytes_per_launch": {"k_clip_fast": 4000}},
               "flops-json": {"flops_per_launch": {"k_clip_fast": 200000},
                              "valu_insts_per_launch": {"k_clip_fast": 8000},
                              "window_units_per_step": {"clip_pairs": 1000.0}}}
    monkeypatch.setattr(bench, "_profile_record", lambda prefix, tag: records[tag])
    n = 1000.0 * share
    assert bench.recorded_traffic("clip") == 4000
    assert bench.recorded_traffic("clip", "clip_pairs", n) == 4000 * share
    flops, insts = bench.recorded_flops("clip", "clip_pairs")
    assert flops * n == 200000 * share and insts * n == 8000 * share
    monkeypatch.setattr(bench, "_profile_record", lambda prefix, tag: None)
    assert bench.recorded_traffic("clip", "clip_pairs", n) is None
    assert bench.recorded_flops("clip", "clip_pairs") is None
