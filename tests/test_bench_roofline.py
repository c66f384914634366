"""The benchmark's roofline figures from a counter record (no GPU)."""
import json
import os

import pytest

import bench


def test_scaled_from_the_counted_launch(monkeypatch):
    """Bytes and operations of a launch that is not the counted one; lanes that sit
    an instruction out do no operation."""
    rec = {"events": 50000, "fetch_kib": 1000.0, "fetch_factor": 2.0, "write_kib": 500.0, "write_factor": 1.0,
           "fp64_flops_per_event": 2e5, "active_lanes": 0.75}
    monkeypatch.setattr(bench, "counters", lambda process: rec)
    same, more = bench.roofline("gg_ttgg", 50000, 1e-3), bench.roofline("gg_ttgg", 262144, 4e-3)
    assert same["traffic"] == pytest.approx(2500 * 1024)
    assert more["traffic"] == pytest.approx(2500 * 1024 * 262144 / 50000)
    assert more["executed_flops_per_event"] == pytest.approx(1.5e5)
    assert more["achieved"] == pytest.approx(1.5e5 * 262144 / 4e-3 / 1e12)
    assert more["frac"] == pytest.approx(more["achieved"] / bench.PEAK["fp64"])


def test_null_without_counters(monkeypatch):
    monkeypatch.setattr(bench, "counters", lambda process: None)
    assert set(bench.roofline("gg_ttgg", 1, 1.0).values()) == {None}


def test_committed_record_is_complete():
    with open(os.path.join(bench.ROOT, "profiles", "counters.json")) as f:
        recs = json.load(f)
    for name, rec in recs.items():
        assert rec["events"] > 0 and 0 < rec["active_lanes"] <= 1, name
        assert {"sources", "fetch_kib", "fetch_factor", "write_kib", "write_factor", "fp64_flops_per_event"} <= set(rec)
