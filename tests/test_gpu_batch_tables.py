"""Batches whose tiling changes between tiled steps: the tables of tiles and of
bands share their memory, and every member stays on the oracle's path."""
import numpy as np
import pytest

import oracle
from paper_1208_2428_amd import Batch, autotune

pytestmark = pytest.mark.gpu

THREADS = oracle.default_threads()
MEMBERS = [dict(width=64 * k, height=34 + 16 * k, seed=70 + k, fill=0.3, force_rate=1e-2, walls=bool(k % 2))
           for k in (1, 2, 5)]


def check(batch):
    batch.sync()
    for m, p in zip(batch.members, MEMBERS):
        ref = oracle.init(p["width"], p["height"], p["seed"], p["fill"], walls=p["walls"])
        ref, _ = oracle.run(ref, 0, m.t, p["seed"], p["force_rate"], threads=THREADS)
        np.testing.assert_array_equal(m.get_state(), ref, err_msg=str((p, m.t)))


@pytest.mark.parametrize("between", ["tiling", "bands", "nothing"])
def test_step_no_deeper_after_the_tables_changed(between):
    b = Batch(MEMBERS)
    b.step(16)
    if between == "bands":
        b.set_tiling(depth=3)
        b.step(7)
    if between == "nothing":
        b.step(0)
    else:
        b.set_tiling()
    for n in (16, 5, 1):
        b.step(n)
    check(b)
    b.close()


@pytest.mark.parametrize("cands", [None, [dict(depth=0, band=0, group_threads=0, passes_per_launch=1)]])
def test_tuned_batch_steps_on(cands, tmp_path, monkeypatch):
    """The tuner's last candidate is the library's own choice; the batch it
    hands back has to step on, whichever candidate won."""
    monkeypatch.setenv("FHP_TUNE_CACHE", str(tmp_path / "tune.json"))
    b = Batch(MEMBERS)
    res = autotune.tune_batch(b, MEMBERS, candidates=cands, steps=16)
    if cands:
        assert res["tiling"] == cands[0]
    for n in (16, 5):
        b.step(n)
    check(b)
    # from the cache as well
    assert autotune.tune_batch(b, MEMBERS, candidates=cands, steps=16)["tiling"] == res["tiling"]
    b.step(16)
    check(b)
    b.close()
