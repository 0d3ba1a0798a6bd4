"""The tiled launch's shapes (one or two copies of a tile, 8 or 12 wavefronts) against one step per
launch, bit for bit: heights on either side of where two copies let two workgroups share a CU,
tile counts on either side of a CU each, cone counts on either side of where a CU each stops
paying, and crowded tiles whose cones fill a part exactly, or one more."""
import numpy as np
import pytest

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu

COEF = ((1.0, 0.01, 1.0), (0.5, 0.02, -1.0))
CASES = [  # grid, cones, crowded, species, depth, height
    ((300, 260), 800, False, 1, 12, 71), ((300, 260), 800, False, 1, 12, 72),
    ((300, 260), 800, False, 2, 12, 71), ((150, 140), 512, True, 1, 10, 64),
    ((150, 140), 513, True, 1, 10, 64), ((300, 260), 512, True, 1, 12, 100),
    ((300, 260), 513, True, 1, 12, 100), ((300, 260), 1536, True, 1, 12, 100),
    ((300, 260), 2304, False, 1, 12, 100), ((300, 260), 2305, False, 1, 12, 100),
    ((300, 260), 1537, True, 2, 12, 70), ((301, 260), 5000, True, 1, 16, 110),
    ((1000, 1300), 3000, False, 1, 12, 70), ((1000, 1300), 3000, False, 1, 12, 150),
    ((1400, 1300), 3000, False, 1, 12, 60),
]


@pytest.mark.parametrize("n,cones,crowd,species,depth,height", CASES)
def test_shapes(n, cones, crowd, species, depth, height):
    sc = S.make_scenario("tile shapes", 2, n, 1.0, 0.2, COEF[:species], 70, (0.5, 2.0), cones, 80,
                         seed=9)
    if crowd:   # every cone starts inside one tile's core
        sc.cone_pos = np.asarray(sc.cone_pos * 0.05 + 40.0, np.float32).astype(np.float64)
    sc.tile = (2, height)
    states = []
    for block in (1, depth):
        with B.Simulation(sc, block_steps=block) as sim:
            if block > 1:
                t = sim.tiling()
                print(f"[gpu] {n} cones={cones} crowded={crowd} {t}", flush=True)
                assert (t["block_steps"], t["height"]) == (depth, height)
            sim.step(depth).step(1)
            sim.counts()
            sim.step(30)
            states.append([sim.field(s) for s in range(species)] +
                          [v for _, v in sorted(sim.cones().items())])
    for a, b in zip(*states):
        np.testing.assert_array_equal(b, a)


def test_recorded_run_with_two_copies():
    sc = S.make_scenario("tile shapes", 2, (260, 240), 1.0, 0.2, COEF, 12, (0.5, 2.0), 1600, 40,
                         seed=10)
    M, out = sc.n_cones, []
    for tile, depth in (((0, 0), 1), ((2, 64), 12), ((2, 70), 12)):
        sc.tile = tile
        with B.Simulation(sc, block_steps=depth) as sim:
            out.append([np.array(sim.adjoint(41, np.arange(M) % 40, np.ones(M), 20))] +
                       [np.array(v) for v in sim.adjoint_backward()])
    for other in out[1:]:
        for a, b in zip(out[0], other):
            np.testing.assert_allclose(b, a, rtol=1e-12)   # the same states; FP64 sums
