"""Host checks that bench.py prices a launch with the counters of launches of
the same kernel, tiles and steps only."""
import json
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

HELD = ["plain", "plain_20_steps", "probe_blocked", "batched_blocked"]


def record(which, tmp_path, monkeypatch, **fields):
    """A record of this workload that belongs to the sources as they are."""
    d = {"kernel_sha256_16": bench.kernel_hash(), "steps_per_launch": 32, "sites_per_lane": 16,
         "extra_sites": 32, "bytes_per_launch": 1000.0, "sq_insts_valu_per_dispatch": 6.144e8, **fields}
    path = tmp_path / (which + ".json")
    path.write_text(json.dumps(d))
    monkeypatch.setitem(bench.TRAFFIC_FILES, which, str(path))


def plan(steps=32, lane=16, extra=32):
    return {"launches": 1, "steps_per_launch": steps, "sites_per_lane": lane, "extra_sites": extra}


def test_a_record_serves_its_plan_only(tmp_path, monkeypatch):
    record("plain", tmp_path, monkeypatch)
    record("plain_20_steps", tmp_path, monkeypatch, steps_per_launch=20, extra_sites=24,
           bytes_per_launch=500.0)
    assert bench.measured_traffic("plain", 32, plan()) == 1000.0
    assert bench.measured_traffic("plain", 20, plan(20, 16, 24)) == 500.0
    # 6.144e8 instructions take 1 ms at 614.4 G/s
    assert bench.valu_issue_frac("plain", 2e-3, 32, plan()) == pytest.approx(0.5)
    for other in (plan(lane=24), plan(extra=40), plan(20, 16, 32), plan(31)):
        assert bench.measured_traffic("plain", other["steps_per_launch"], other) is None


def test_no_record_of_other_sources(tmp_path, monkeypatch):
    record("plain", tmp_path, monkeypatch, kernel_sha256_16="0" * 16)
    assert bench.measured_traffic("plain", 32, plan()) is None


def test_roofline_of_a_plan_nobody_counted(tmp_path, monkeypatch):
    record("plain", tmp_path, monkeypatch)
    record("plain_20_steps", tmp_path, monkeypatch, steps_per_launch=20)
    r = bench.roofline(5000.0, 0.03, plan(24))
    assert r["bound"] == "alu" and r["frac"] is None and r["achieved"] is None and r["traffic"] is None
    assert r["at_12_bytes_per_update"]["frac"] == pytest.approx(5000.0 / bench.HBM_PEAK_GBS)
    r = bench.roofline(5000.0, 0.03125, plan())
    assert r["frac"] == pytest.approx(1.0) and r["traffic"] == 1000.0
    one = bench.roofline(5000.0, 0.03, plan(1, 0, 0))
    assert one["bound"] == "hbm" and one["frac"] == pytest.approx(5000.0 / bench.HBM_PEAK_GBS)


@pytest.mark.parametrize("which", HELD)
def test_records_name_their_plan(which):
    d = json.load(open(bench.TRAFFIC_FILES[which]))
    assert d["sites_per_lane"] in (4, 8, 16, 24) and d["extra_sites"] % 8 == 0
    assert d["steps_per_launch"] > 1


def test_20_step_record_follows_from_its_counters():
    d = json.load(open(bench.TRAFFIC_FILES["plain_20_steps"]))
    cal = d["copy_calibration"]
    want = 1024 * (d["fetch_size_kib_per_dispatch"] * cal["fetch_factor"] +
                   d["write_size_kib_per_dispatch"] * cal["write_factor"])
    assert d["bytes_per_launch"] == pytest.approx(want, rel=1e-9)
    assert d["steps_per_launch"] == 20
    assert d["algorithmic_bytes_per_launch"] == bench.BYTES_PER_SITE_UPDATE * (1 << 24) * 20


def test_d2q9_record_covers_the_lattice():
    v = json.load(open(bench.D2Q9_TILES_FILE))
    assert v["sites"] == 4096 * 4096
    # a wave takes 64 sites of several tiles
    assert (v["sites"] // 64) % v["sq_waves_per_dispatch"] == 0
    assert [os.path.basename(p) for p in bench.D2Q9_SRCS] == v["kernel_sources"]
