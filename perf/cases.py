"""The work this library is measured on: what its users have it do, through its
public entry points, from the smallest lattice to the largest.

Every case has a ``kind``, the way a program uses the library:

  step    a simulation that is kept: advance it, read what is asked for (row
          sums for a velocity profile) and the state (byte per node);
  sweep   a short simulation made, run, read and closed in one go, as in a
          parameter sweep;
  field   a device-resident lattice advanced by ``fhp_step_noalloc`` from one
          tensor to another;
  resume  a state taken in from the host, all its observables, the state back
          out (checkpoint, analysis);
  batch   uneven lattices advanced together, 16 x 16 block fields of each;
  jobs    a pool that is kept open: jobs of uneven sizes and lengths admitted,
          ticked to their ends, their block fields read.

All outputs are whole numbers: there is one correct result, bit for bit.
"""
from __future__ import annotations

import ctypes
import functools
import math
import random

import numpy as np
import torch

from paper_1208_2428_amd import Batch, Pool, Sim
from paper_1208_2428_amd import _binding as B
from paper_1208_2428_amd import workloads as WL

BLOCK = 16  # nodes per side of a block of the density and momentum fields


def listed() -> list[dict]:
    def step(name, W, H, steps, fill, force=0.0, walls=False, mask=0.0, rules=B.RULES_FHP2,
             rows=False):
        return dict(name=name, kind="step", width=W, height=H, steps=steps, fill=fill, force=force,
                    walls=walls, mask=mask, rules=rules, rows=rows)

    return [
        # The smallest call: a short channel of 5-word rows advanced by a few
        # steps inside a loop that may not allocate.  Latency alone.
        dict(name="field-320x96", kind="field", width=320, height=96, steps=12, fill=0.25,
             force=1e-3, walls=True, rules=B.RULES_FHP2),
        # The small periodic box without forcing, 1000 steps (workload torus-256).
        step("torus-256", 256, 256, 1000, 0.2),
        # One point of a parameter sweep on short channels: set-up, a short
        # run, the velocity profile and the state.
        dict(name="sweep-1024x512", kind="sweep", width=1024, height=512, steps=200, fill=0.25,
             force=1e-3, walls=True, mask=0.0, rules=B.RULES_FHP2, rows=True),
        # A duct with obstacles whose rows are 31 words: no power of two, no
        # full wave, heights that no band divides.
        step("duct-1984x1030", 1984, 1030, 600, 0.3, 1e-3, True, 0.05, rows=True),
        # FHP-I on a square box with forcing: the six-velocity model.
        step("fhp1-2048", 2048, 2048, 600, 0.2, 5e-4, rules=B.RULES_FHP1),
        # FHP-III (collision-saturated, the least viscous model) round obstacles.
        step("fhp3-4096x2048", 4096, 2048, 600, 0.25, 5e-4, True, 0.05, rules=B.RULES_FHP3),
        # The Poiseuille channel of the workloads, a fifth of its run, with
        # its velocity profile.
        step("channel-4096", 4096, 4096, 2000, 0.25, 1e-3, True, rows=True),
        # A device-resident periodic lattice near the largest state that the
        # allocation-free call takes; rows of two waves.
        dict(name="field-8192x8128", kind="field", width=8192, height=8128, steps=300, fill=0.3,
             force=5e-4, walls=False, rules=B.RULES_FHP2),
        # The headline: the 16384^2 porous medium, run on between two
        # checkpoints.
        step("porous-16384", 16384, 16384, 6000, 0.3, 5e-4, False, 0.05),
        # Analysis of a saved state of ragged size with obstacles.
        dict(name="resume-4032x4090", kind="resume", width=4032, height=4090, fill=0.3, force=5e-4,
             walls=True, mask=0.05),
        # An ensemble of uneven periodic lattices, 500 steps each, drawn as
        # the ensemble workload draws its 512.
        dict(name="ensemble-60", kind="batch", members=60, lmin=128, lmax=2048, steps=500,
             force=0.0),
        # A burst of channel-flow jobs served by a pool, drawn as the request
        # stream draws them, on sides up to 4096.
        dict(name="jobs-32", kind="jobs", jobs=32, lmin=256, lmax=4096, smin=100, smax=2000),
    ]


# A drawn case's node updates stay below this (the largest listed case has 1.6e12).
MOST_UPDATES = 3e11


def draw(rng: random.Random) -> dict:
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def size(wmax, hmax, nodes):
        """Widths of 1 word up, any word count; heights even; at most `nodes` nodes."""
        while True:
            W, H = 64 * log_int(1, wmax // 64), 2 * log_int(4, hmax // 2)
            if W * H <= nodes:
                return W, H

    def steps(W, H, lo, hi):
        return max(lo, min(log_int(lo, hi), int(MOST_UPDATES / (W * H))))

    kind = rng.choice(["step", "step", "step", "sweep", "field", "field", "resume", "batch", "jobs"])
    fill = round(rng.uniform(0.1, 0.4), 3)
    force = rng.choice([0.0, 1e-3, 5e-4, round(rng.uniform(1e-5, 5e-3), 6)])
    walls = rng.random() < 0.5
    if kind in ("step", "sweep"):
        W, H = size(16384, 16384, 2**28) if kind == "step" else size(2048, 2048, 2**21)
        mask = 0.05 if min(W, H) >= 128 and W * H <= 2**24 and rng.random() < 0.5 else 0.0
        return dict(kind=kind, width=W, height=H,
                    steps=steps(W, H, 100, 2000) if kind == "step" else log_int(50, 500), fill=fill,
                    force=force, walls=walls, mask=mask,
                    rules=rng.choice([B.RULES_FHP2, B.RULES_FHP2, B.RULES_FHP1, B.RULES_FHP3]),
                    rows=rng.random() < 0.5)
    if kind == "field":
        W, H = size(8192, 8192, 2**26)
        return dict(kind=kind, width=W, height=H, steps=steps(W, H, 5, 500), fill=fill, force=force,
                    walls=walls, rules=rng.choice([B.RULES_FHP2, B.RULES_FHP2, B.RULES_FHP1, B.RULES_FHP3]))
    if kind == "resume":
        W, H = size(4096, 4096, 2**24)
        return dict(kind=kind, width=W, height=H, fill=fill, force=force, walls=walls,
                    mask=0.05 if min(W, H) >= 128 and rng.random() < 0.5 else 0.0)
    if kind == "batch":
        lmax = 64 * rng.randint(4, 32)
        return dict(kind=kind, members=rng.randint(4, 60), lmin=128, lmax=lmax,
                    steps=log_int(50, 500), force=rng.choice([0.0, 1e-3]))
    return dict(kind=kind, jobs=rng.randint(4, 32), lmin=256, lmax=64 * rng.randint(8, 64), smin=100,
                smax=log_int(200, 2000))


@functools.lru_cache(maxsize=4)
def disks(W: int, H: int, frac: float) -> np.ndarray:
    """The obstacles of a W x H case: a program's geometry, the same in all its runs."""
    r = max(2, min(32, min(W, H) // 16))
    return WL.porous_mask(W, H, 33, max(1, r // 4), r, frac)


def sim_params(case: dict, seed: int) -> dict:
    return dict(width=case["width"], height=case["height"], seed=seed, fill=case["fill"],
                force_rate=case["force"], walls=case["walls"],
                solid=disks(case["width"], case["height"], case["mask"]) if case.get("mask") else None,
                rules=case.get("rules", B.RULES_FHP2))


def members(case: dict, seed: int) -> list[dict]:
    """The case's members; the sizes belong to the case, seeds and densities to the seed."""
    rng = np.random.default_rng(seed)
    return [dict(width=m.width, height=m.height, seed=int(rng.integers(0, 2**63)),
                 fill=float(rng.uniform(0.1, 0.4)), force_rate=case["force"])
            for m in WL.batch_members(n=case["members"], seed=4, lmin=case["lmin"], lmax=case["lmax"])]


def requests(case: dict) -> list[WL.Request]:
    return WL.request_stream(n=case["jobs"], seed=5, side_lo=case["lmin"], side_hi=case["lmax"],
                             steps_lo=case["smin"], steps_hi=case["smax"])


def job_words(side: int) -> int:
    """Arena words of one job: two buffers of seven planes and an obstacle plane."""
    return 15 * ((side * side // 64 + 31) // 32 * 32)


def prepare(case: dict, seed: int) -> dict:
    kind = case["kind"]
    if kind == "step":
        return dict(case=case, sim=Sim(**sim_params(case, seed)))
    if kind == "sweep":
        return dict(case=case, params=sim_params(case, seed))
    if kind == "field":
        W, H, dev = case["width"], case["height"], torch.device("cuda", torch.cuda.current_device())
        g = torch.Generator(device=dev)
        g.manual_seed(seed)
        # every channel bit set with probability `fill`, to six binary digits
        planes = torch.zeros(7, H, W // 64, dtype=torch.int64, device=dev)
        for digit in range(6, 0, -1):
            word = torch.randint(-2**63, 2**63 - 1, planes.shape, dtype=torch.int64, device=dev,
                                 generator=g)
            planes = planes | word if int(case["fill"] * 2**digit) & 1 else planes & word
        params, _ = B.make_params(W, H, seed=seed, force_rate=case["force"], walls=case["walls"],
                                  rules=case["rules"])
        return dict(case=case, lib=B.load(), params=params, src=planes, dst=torch.empty_like(planes))
    if kind == "resume":
        p = sim_params(case, seed)
        rng = np.random.default_rng(seed)
        state = np.zeros((p["height"], p["width"]), dtype=np.uint8)
        level = int(round(case["fill"] * 256))
        for c in range(7):
            state |= (rng.integers(0, 256, state.shape, dtype=np.uint8) < level).astype(np.uint8) << c
        if p["solid"] is not None:
            state[p["solid"] != 0] = 0x80
        return dict(case=case, sim=Sim(**p), state=state)
    if kind == "batch":
        return dict(case=case, batch=Batch(members(case, seed)))
    reqs = requests(case)
    rng = np.random.default_rng(seed)
    jobs = [(r.steps, dict(width=r.side, height=r.side, seed=int(rng.integers(0, 2**63)), fill=r.fill,
                           force_rate=r.force_rate, walls=r.walls)) for r in reqs]
    slots = len(jobs)
    bands = sum(r.side // 2 for r in reqs)
    arena = Pool.arena_bytes_for(slots, bands, 8 * sum(job_words(r.side) for r in reqs))
    return dict(case=case, jobs=jobs, pool=Pool(arena, max_slots=slots, max_bands=bands,
                                                group_threads=256))


def run(state: dict):
    case = state["case"]
    kind = case["kind"]
    if kind == "step":
        sim = state["sim"]
        sim.step(case["steps"])
        out = {"state": sim.get_state()}
        if case["rows"]:
            out["rows"] = sim.observe_rows()
        return out
    if kind == "sweep":
        sim = Sim(**state["params"])
        sim.step(case["steps"])
        out = {"state": sim.get_state()}
        if case["rows"]:
            out["rows"] = sim.observe_rows()
        sim.close()
        return out
    if kind == "field":
        stream = torch.cuda.current_stream(state["src"].device)
        B.check(state["lib"].fhp_step_noalloc(
            ctypes.byref(state["params"]), ctypes.c_void_p(state["src"].data_ptr()),
            ctypes.c_void_p(state["dst"].data_ptr()), None, 0, case["steps"], 0,
            ctypes.c_void_p(stream.cuda_stream)))
        return state["dst"]
    if kind == "resume":
        sim = state["sim"]
        sim.set_state(state["state"], t=1000)
        total = sim.observe_global()
        return {"total": np.array([total["mass"], total["px"], total["py"], *total["channels"], total["solid"]]),
                "rows": sim.observe_rows(), "blocks": sim.observe_blocks(BLOCK),
                "digest": np.array([sim.digest()], dtype=np.uint64).view(np.int64),
                "state": sim.get_state()}
    if kind == "batch":
        batch = state["batch"]
        batch.step(case["steps"])
        batch.sync()
        return [m.observe_blocks(BLOCK) for m in batch.members]
    pool, jobs = state["pool"], state["jobs"]
    slot_job = {pool.admit(steps, **params): j for j, (steps, params) in enumerate(jobs)}
    fields = [None] * len(jobs)
    while slot_job:
        pool.tick()
        for slot in pool.done():
            fields[slot_job.pop(slot)] = pool.result(slot, BLOCK)
            pool.release(slot)
    return fields


def work(case: dict) -> dict:
    """Bytes: seven planes (and the obstacles) read once and written once per
    call, the host's bytes and the fields; flops: two 32-bit lane operations a
    node and step, about what the collision and the random words take when 32
    nodes share a word."""
    kind = case["kind"]
    if kind in ("batch", "jobs"):
        parts = [(m["width"] * m["height"], case["steps"]) for m in members(case, 0)] if kind == "batch" \
            else [(r.side * r.side, r.steps) for r in requests(case)]
        nodes = sum(n for n, _ in parts)
        return {"bytes": nodes * (14 / 8 + 12 / BLOCK**2), "flops": 2.0 * sum(n * s for n, s in parts)}
    nodes = case["width"] * case["height"]
    state = nodes * (7 + bool(case.get("mask"))) / 8
    if kind == "field":
        return {"bytes": 2 * state, "flops": 2.0 * nodes * case["steps"]}
    if kind == "resume":
        return {"bytes": 2 * nodes + state + nodes * 12 / BLOCK**2 + 24 * case["height"],
                "flops": 2.0 * nodes}
    rows = 24 * case["height"] if case["rows"] else 0
    return {"bytes": nodes + (2 if kind == "step" else 1) * state + rows,
            "flops": 2.0 * nodes * case["steps"]}


def exact(case: dict, seed: int):
    """No output is a rounded number: every one is a whole number with one
    correct value."""
    return None
