"""Un-blocked steps whose cones share a launch with the next field step, against the same steps
asked for one at a time (each part then has a launch of its own) and with launches timed.  Every
cell and cone is updated by the same expressions either way, so the states are equal bit for
bit."""
import numpy as np
import pytest

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu

COEF = ((1.0, 0.01, 1.0), (0.5, 0.02, -1.0))
CASES = [  # grid, cones, species: ragged boxes, one cone, one workgroup's cones and one more
    ((33, 21), 1, 1), ((257, 9), 256, 2), ((300, 65), 257, 1), ((700, 130), 5000, 2),
    ((3, 3, 3), 1, 1), ((65, 9, 5), 512, 2), ((64, 8, 8), 513, 1), ((70, 40, 33), 4097, 2),
    ((130, 70, 90), 30000, 1), ((40, 30, 20), 70001, 1),
]


def _state(sim, n_species):
    c = sim.cones()
    return [sim.field(s) for s in range(n_species)] + [c[k] for k in sorted(c)]


@pytest.mark.parametrize("n,cones,species", CASES)
def test_shared_launches_leave_the_same_state(n, cones, species):
    print(f"[gpu] {n} cones={cones} species={species}", flush=True)
    sc = S.make_scenario("launches", len(n), n, 1.0, 0.12, COEF[:species], 3, (0.5, 2.0), cones,
                         40, seed=3)
    steps = 70   # crosses two refreshes of the 3D order
    with B.Simulation(sc, block_steps=1) as one:
        for _ in range(steps):
            one.step(1)
        want = _state(one, species)
    with B.Simulation(sc, block_steps=1) as sim:
        sim.step(steps)
        got = _state(sim, species)
    with B.Simulation(sc, block_steps=1) as sim:   # reads and refreshes in between, timed steps
        sim.step(5)
        sim.cones()
        B.sim_set_timing(sim.h, True)
        sim.step(2)
        B.sim_set_timing(sim.h, False)
        sim.step(steps - 7)
        mixed = _state(sim, species)
    for w, g, x in zip(want, got, mixed):
        np.testing.assert_array_equal(g, w)
        np.testing.assert_array_equal(x, w)
