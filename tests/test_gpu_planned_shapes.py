"""Planned launch shapes (depth and tile heights, of one simulation and of a batch) against one
step per launch: the same expressions in the same order for every cell and cone, so the states
are equal bit for bit.  Long steps leave little or no core at the deeper shapes, one-row and
one-tile grids sit at the other end, and uneven batches mix both."""
import copy

import numpy as np
import pytest

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu

COEF = ((1.0, 0.01, 1.0), (0.5, 0.02, -1.0))


def _case(n, cones, species, step_len, seed):
    return S.make_scenario("shapes", 2, n, 1.0, 0.2, COEF[:species], 5, (0.5, 2.0), cones, 12,
                           step_len=step_len, seed=seed, sim_index=seed)


def _state(cones, fields):
    return [cones[k] for k in sorted(cones)] + fields


def _alone(sc, steps):
    with B.Simulation(sc, block_steps=1) as sim:
        sim.step(steps)
        return _state(sim.cones(), [sim.field(s) for s in range(len(sc.species))])


def _same(got, want):
    for g, w in zip(got, want):
        np.testing.assert_array_equal(g, w)


@pytest.mark.parametrize("n,cones,species,step_len,hint", [
    ((5, 3), 7, 1, 0.5, 0), ((640, 2), 50, 2, 0.5, 0), ((3, 500), 60, 1, 0.5, 0),
    ((128, 128), 600, 1, 0.0, 0), ((300, 210), 900, 2, 2.0, 0), ((300, 210), 900, 1, 4.5, 0),
    ((200, 150), 300, 1, 12.0, 0), ((200, 150), 300, 1, 0.5, 110), ((90, 700), 300, 2, 0.5, 64),
])
def test_default_depth(n, cones, species, step_len, hint):
    print(f"[gpu] {n} step {step_len} height {hint}", flush=True)
    sc = _case(n, cones, species, step_len, 4)
    sc.tile = (0, hint)
    with B.Simulation(sc) as sim:
        sim.step(1).step(39)
        got = _state(sim.cones(), [sim.field(s) for s in range(species)])
    _same(got, _alone(sc, 40))


BATCHES = [  # sizes, cones each, species, step length, depth asked for, height hint of the first
    ([(5, 3), (64, 64), (511, 40)], 70, 1, 0.5, 0, 0),
    ([(64 + 37 * k, 500 - 41 * k) for k in range(9)], 200, 1, 0.5, 0, 0),
    ([(150, 150)] * 24, 300, 2, 0.5, 0, 0), ([(150, 150)] * 3, 3000, 1, 0.5, 8, 0),
    ([(90, 80), (200, 333)], 100, 1, 3.0, 0, 0), ([(90, 80), (200, 333)], 100, 1, 0.5, 12, 80),
]


@pytest.mark.parametrize("sizes,cones,species,step_len,depth,hint", BATCHES)
def test_batch(sizes, cones, species, step_len, depth, hint):
    print(f"[gpu] batch of {len(sizes)}, step {step_len}, depth {depth}", flush=True)
    scs = [_case(n, cones, species, step_len, 10 + i) for i, n in enumerate(sizes)]
    scs[0].tile = (0, hint)
    bt = B.Batch([copy.copy(sc) for sc in scs], graph_launches=2, block_steps=depth)
    bt.step(37)
    for i, sc in enumerate(scs):
        got = _state(bt.cones(i), [bt.field(i, s) for s in range(species)])
        _same(got, _alone(sc, 37))
    bt.close()
