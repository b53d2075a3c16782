"""A tuning cache written among other candidates: its entries (no set of
candidates in their keys) are kept in the file and not taken."""
import json

import pytest

from paper_2405_00814_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_choices_among_other_candidates(tmp_path, monkeypatch):
    from paper_2405_00814_amd.sim import Batch, Sim
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("GEMFDTD_TUNE_CACHE", str(cache))
    pb = W.dielectric2d(160, ny=192, steps=60, seed=3, nrect=6, side=(6, 30), npml=8, nprobes=3)
    probs = W.batch2d(count=3, steps=0, seed=5, side=(70, 120), nprobes=2, rect_side=(8, 40), rect_density=40.0 / 4096)
    s, b = Sim.from_problem(pb), Batch(probs)
    s.autotune(8)
    b.autotune(8)
    keys = list(json.loads(cache.read_text()))
    assert len(keys) == 2
    # the slowest configurations under keys of a former form
    old = {k.rsplit("|", 1)[0]: [1, 1, 1, 0] if "|batch|" in k else [1, 0, 0, 0, 0, 1] for k in keys}
    cache.write_text(json.dumps(old))
    assert s.autotune(8)["variant"] != 1
    assert b.autotune(8)[0] != 1
    now = json.loads(cache.read_text())
    assert set(now) == set(old) | set(keys) and all(now[k] == v for k, v in old.items())
    s.close()
    b.close()
