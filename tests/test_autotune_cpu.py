"""The autotuner's cache file (no GPU: the sweeps are replaced by tables of their results)."""
import json

import pytest

import workloads as W
from paper_0907_4027_amd import autotune

SINGLE = {"pixels_per_lane": 0, "segment": 0, "traps_per_lane": 0, "rows": 0, "iteration_us": 7.0}
BATCH = {"traps_per_lane": 0, "rows": 0, "pixels_per_lane": 0, "ms_per_solve": 0.2}


class FakeContext:
    def __init__(self):
        self.knobs = None

    def set_tuning(self, **knobs):
        self.knobs = knobs


@pytest.mark.parametrize("batched", [False, True])
def test_entries_of_other_kernels_are_measured_again(monkeypatch, tmp_path, batched):
    """An entry written before the tile kernels (no "kernels" name, a direct-sum knob in it) is not applied;
    the entry that replaces it is, without another sweep, and other entries of the file stay."""
    best, sweeps = dict(BATCH if batched else SINGLE), []

    def sweep(*a, **k):
        sweeps.append(1)
        return [best]

    for name in ("cache_key", "batch_key"):
        monkeypatch.setattr(autotune, name, lambda *a, **k: "here")
    for name in ("sweep", "sweep_batched"):
        monkeypatch.setattr(autotune, name, sweep)
    old = best | {"pixels_per_lane": 1, "rows": 1}
    path = tmp_path / "tuning.json"
    path.write_text(json.dumps({"here": old, "there": old}))
    slm, xyz = W.Slm(64, 64), [[0.0, 0.0, 0.0]] * 3
    for turn in range(2):
        c = FakeContext()
        if batched:
            r = autotune.tune_batched(c, slm, [1, 2], xyz, [0.0] * 3, cache=str(path))
        else:
            r = autotune.tune(c, slm, xyz, [0.0] * 3, cache=str(path))
        assert set(c.knobs.values()) == {0} and r["knobs"] == c.knobs
        assert (r["table"] is None) == (turn == 1)
    assert len(sweeps) == 1
    db = json.loads(path.read_text())
    assert db["there"] == old and db["here"]["kernels"] == autotune.KERNELS
