"""The gradient on a grid of so many reverse tiles that a launch over them takes two slices: the cue
and the cones lie at its left end, so that it equals the gradient on a grid of 2000 columns."""
import numpy as np
import pytest

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu


def test_two_slices_of_tiles():
    out = []
    for nx in (2000, 120_000_000):   # 1,071,429 tiles
        print(f"[gpu] {nx} x 2", flush=True)
        sc = S.make_scenario("wide", 2, (2000, 2), 1.0, 0.15, ((1.0, 0.01, 1.0),), 6, (0.5, 2.0), 40,
                             8, step_len=0.05, seed=3)
        at = np.arange(6) * 7 + 300
        sc.species[0].source_cell = (at + nx * (np.arange(6) % 2)).astype(np.int32)
        sc.cone_pos[:, 0] = np.linspace(298.0, 340.0, 40, dtype=np.float32)
        sc.nx, sc.turn_gain = nx, 0.2
        with B.Simulation(sc, block_steps=1) as sim:
            loss = sim.adjoint(13, np.arange(40) % 8, np.linspace(0.5, 1.5, 40), 5)
            out.append([np.array(loss)] + [np.array(v) for v in sim.adjoint_backward()])
            sim.step(2)
    for narrow, wide in zip(*out):
        assert np.all(narrow != 0)
        np.testing.assert_array_equal(wide, narrow)
