"""The tuner keeps the library's own choice where no named tiling beats it, and
the committed table holds no tiling that lost to it."""
import os

import pytest
import torch

from paper_1905_04582_amd import autotune

TABLE = autotune.load(os.path.join(os.path.dirname(autotune.__file__), "tuning.json"))
SINGLE = sorted(k for k in TABLE if not k.startswith("batch|"))


def test_choose():
    assert autotune.choose((64, 2), 1.0, 1.5) == (64, 2)
    assert autotune.choose((64, 2), 1.0, 1.0) == (0, 0)
    assert autotune.choose((64, 2), 0.995, 1.0) == (0, 0)      # within the margin
    assert autotune.choose((64, 2), 1.5, 1.0) == (0, 0)


@pytest.mark.parametrize("key", SINGLE)
def test_committed_entry_beats_the_default(key):
    e = TABLE[key]
    want = autotune.choose((e["tile_rows"], e["tile_waves"]), e["best_in_turn_ms"],
                           e["default_in_turn_ms"])
    assert (e["tile_rows"], e["tile_waves"]) == want


def test_default_entry_is_looked_up(tmp_path, monkeypatch):
    monkeypatch.setenv("MDS_TUNE_CACHE", str(tmp_path / "t.json"))
    monkeypatch.setattr(autotune, "_arch", lambda device=None: "gfx950")
    autotune.save({autotune._key("gfx950", torch.float64, 2, 1000): dict(
        tile_rows=0, tile_waves=0, best="8x64/1", ms=1.0)})
    assert autotune.lookup(torch.float64, 2, 1000) == (0, 0)
