"""Cached pool tunings: a choice made when time_block 2 with the default
time_rows still meant sweeps of 16 rows is not used, and those sweeps are a
candidate of their own."""
import json

from paper_2303_08163_amd import autotune


def test_choices_among_other_kernels_are_not_used(monkeypatch, tmp_path):
    monkeypatch.setattr(autotune, "_device_key", lambda: "test-device")
    doms = [(9, (40, 50), "fp32_dev")]
    cache = tmp_path / "tune.json"
    old = dict(tile_x=16, tile_y=4, persistent=0)
    cache.write_text(json.dumps({f"candidates-v9|test-device|{autotune.signature(doms)}": {"tuning": old}}))
    blocks = dict(tile_x=64, tile_y=4, persistent=0, row_fit=1, time_block=2, time_rows=0)
    monkeypatch.setattr(autotune, "time_tuning", lambda d, c, steps=60: 1e-3 if c == blocks else 2e-3)
    best, rep = autotune.tune_pool(doms, cache_path=str(cache))
    assert best == blocks and not rep["cached"]
    assert autotune.tune_pool(doms, cache_path=str(cache))[1]["cached"]


def test_every_sweep_length_is_a_candidate():
    launch = [c for c in autotune.candidates() if c.get("time_block") == 2 and c["persistent"] == 0]
    assert sorted(c["time_rows"] for c in launch) == [0, 16, 32, 64]
