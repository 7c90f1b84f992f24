"""What the tuner's disk cache and candidate list depend on: entries timed on
other kernels are not taken, plans of one shape whose steps have other passes
do not share an entry, and no launch sequence is timed twice."""
import json
import os

import numpy as np
import pytest

from paper_2609_08384_amd import autotune, brahms


@pytest.fixture
def tuner(monkeypatch, tmp_path):
    monkeypatch.setenv("BRAHMS_CACHE_DIR", str(tmp_path))
    monkeypatch.setattr(autotune, "_arch", lambda device: "gfx950")
    autotune._memo.clear()
    calls = []

    def measure(nx, ny, nt, nf, params, schedule, device="cuda:0", steps=64, warmup=3):
        calls.append(dict(schedule))
        return 1.0 + schedule["pass_order"]
    monkeypatch.setattr(autotune, "measure", measure)
    yield calls, os.path.join(str(tmp_path), "schedules.json")
    autotune._memo.clear()


def _params(alpha=0.0):
    return brahms.Params(dz=0.01, fields=[brahms.FieldParams(kappa=1.0, alpha=alpha)] * 2)


def test_entries_of_other_kernels_are_timed_again(tuner):
    calls, path = tuner
    stale = {"pass_order": 3, "graph": 0, "merge_halves": 1, "fuse_steps": 0}
    with open(path, "w") as fh:
        json.dump({"v8:gfx950:32x32x32:nf2:m1": {"schedule": stale, "ms_per_step": 1.0}}, fh)
    best = autotune.tune(32, 32, 32, 2, _params())
    assert calls and best["pass_order"] == 0
    autotune._memo.clear()
    calls.clear()
    assert autotune.tune(32, 32, 32, 2, _params()) == best and not calls


def test_lossy_and_lossless_cw_plans_do_not_share_an_entry(tuner):
    calls, path = tuner
    autotune.tune(64, 64, 1, 2, _params())
    calls.clear()
    autotune.tune(64, 64, 1, 2, _params(alpha=0.1))
    assert calls
    mapped = _params()
    mapped.dk_map = np.zeros((64, 64))
    autotune.tune(64, 64, 1, 2, mapped)
    with open(path) as fh:
        assert len(json.load(fh)) == 3


def test_two_axis_steps_are_timed_once(tuner):
    calls, _ = tuner
    autotune.tune(64, 48, 1, 2, _params())
    timed = calls[1:]   # (the first is a warm-up)
    assert all(c["fuse_steps"] == 0 and c["pass_order"] < 2 and not c.get("wide") for c in timed)
    assert {(c["pass_order"], c["graph"]) for c in timed} == {(o, g) for o in (0, 1) for g in (0, 1)}
