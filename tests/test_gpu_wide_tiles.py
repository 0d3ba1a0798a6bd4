"""Tall tiles of four-column segments, stepped by sixteen wavefronts, against one step per launch
bit for bit: at the height where sixteen take over from eight and at the tallest, with tiles
that no, one or several further parts of 1024 cones share, with ragged grids and unaligned rows,
under the SNR law, and recording a run for the gradient."""
import numpy as np
import pytest

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu


def _case(n, cones, crowd, seed=6):
    sc = S.make_scenario("wide", 2, n, 1.0, 0.2, ((1.0, 0.01, 1.0),), 80, (0.5, 2.0), cones, 90,
                         seed=seed)
    if crowd:   # every cone starts inside one tile's core
        sc.cone_pos = np.asarray(sc.cone_pos * 0.05 + 40.0, np.float32).astype(np.float64)
    return sc


def _state(sim):
    return dict(sim.cones(), field=sim.field())


CASES = [  # grid, cones, crowded, depth, height
    ((512, 300), 3000, False, 14, 95), ((512, 300), 3000, False, 14, 96),
    ((509, 301), 700, False, 12, 130), ((1023, 77), 50, False, 16, 143),
    ((400, 390), 1023, True, 14, 134), ((400, 390), 1024, True, 14, 134),
    ((400, 390), 1025, True, 14, 134), ((401, 390), 5000, True, 10, 150),
]


@pytest.mark.parametrize("n,cones,crowd,depth,height", CASES)
def test_wide_tiles(n, cones, crowd, depth, height):
    print(f"[gpu] {n} cones={cones} crowded={crowd} depth={depth} height={height}", flush=True)
    sc = _case(n, cones, crowd)
    with B.Simulation(sc, block_steps=1) as sim:
        sim.step(45)
        want = _state(sim)
    sc.tile = (4, height)
    with B.Simulation(sc, block_steps=depth) as sim:
        t = sim.tiling()
        assert (t["block_steps"], t["cols_per_lane"], t["height"]) == (depth, 4, height)
        sim.step(depth).step(3)
        sim.counts()
        sim.step(45 - depth - 3)
        got = _state(sim)
    for k in want:
        np.testing.assert_array_equal(got[k], want[k], err_msg=k)


def test_recorded_run():
    sc = _case((300, 280), 900, True)
    M = sc.n_cones
    out = []
    for tile, depth in (((0, 0), 1), ((4, 130), 12)):
        sc.tile = tile
        with B.Simulation(sc, block_steps=depth) as sim:
            out.append([np.array(sim.adjoint(40, np.arange(M) % 90, np.ones(M), 20))] +
                       [np.array(v) for v in sim.adjoint_backward()])
    for a, b in zip(*out):
        np.testing.assert_allclose(b, a, rtol=1e-12)   # the same states; FP64 sums, in any order
