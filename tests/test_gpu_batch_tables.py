"""Batches and pools whose tables change, or stay, between tiled steps: tiles and
bands share the tables' memory, and every lattice stays on the oracle's path."""
import numpy as np
import pytest
import torch

import oracle
from paper_1208_2428_amd import Batch, Pool, autotune

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


@pytest.mark.parametrize("passes,steps", [(1, 6), (1, 9), (2, 11), (2, 14)])
def test_ended_job_stays_as_it_ended(passes, steps):
    """A job that ended with a remainder of a tick is not stepped again while it
    stays resident beside others: neither buffer changes."""
    W, H = 320, 130
    pool = Pool(Pool.arena_bytes_for(4, 256, 4 << 20), max_slots=4, max_bands=256)
    tables = Pool.arena_bytes_for(4, 256, 0)
    job = dict(width=W, height=H, seed=5, fill=0.3, force_rate=1e-2)
    slot = pool.admit(steps, **job)
    pool.admit(200, **dict(job, seed=6))
    pool.tick(passes)
    assert pool.done() == [slot]
    pool.sync()
    both = slice(tables, tables + 2 * 7 * ((W // 64 * H + 31) // 32 * 32) * 8)
    before = pool.arena[both].clone()
    for _ in range(2):
        pool.tick(passes)
    pool.sync()
    assert torch.equal(pool.arena[both], before)
    ref = oracle.init(W, H, 5, 0.3)
    ref, _ = oracle.run(ref, 0, steps, 5, 1e-2, threads=THREADS)
    np.testing.assert_array_equal(pool.member(slot).get_state(), ref)
    pool.close()
