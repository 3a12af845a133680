"""Calls of a few steps by the default route, on both sides of where it goes from
tiles to sweeping bands, bit for bit against single steps."""
import numpy as np
import pytest

from paper_1208_2428_amd import Sim

pytestmark = pytest.mark.gpu

SHAPES = [(4096, 4096), (4032, 4090), (3456, 4096), (4096, 3442), (4096, 4608), (4096, 2048), (4096, 4610),
          (3584, 3584), (384, 400000), (512, 300002), (4096, 37000)]


@pytest.mark.parametrize("rules", [0, 1, 2])
@pytest.mark.parametrize("W,H", SHAPES)
def test_short_calls_match_single_steps(W, H, rules):
    k = SHAPES.index((W, H))
    solid = (np.random.default_rng(k).random((H, W)) < 0.02).astype(np.uint8) if k % 2 else None
    kw = dict(seed=7 + k, fill=0.3, force_rate=7e-3 * (k % 3), walls=k % 2 == 0, solid=solid, rules=rules)
    a, b = Sim(W, H, **kw), Sim(W, H, **kw, depth=1)
    for n in (2, 3, 4, 2):
        a.step(n)
        b.step(n)
        assert a.digest() == b.digest(), (n, a.t)
    a.close()
    b.close()


@pytest.mark.parametrize("rules", [0, 1, 2])
def test_large_lattice_passes_of_every_depth(rules):
    """Evenly deep passes: single steps, and 4 + 3, 5 + 4 + 4, 6 + 6 + 6 (FHP-III in threes)."""
    kw = dict(seed=11, fill=0.3, force_rate=5e-3, walls=True, rules=rules)
    a, b = Sim(16384, 9282, **kw), Sim(16384, 9282, **kw, depth=1)
    for n in (1, 7, 13, 18):
        a.step(n)
        b.step(n)
        assert a.digest() == b.digest(), (n, a.t)
    a.close()
    b.close()
