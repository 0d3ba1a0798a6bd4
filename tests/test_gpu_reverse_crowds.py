"""Reverse launches over tiles with more cones than are held in LDS: grids crowded on the whole (a
thread per further cone) and grids with a crowd in one place (four), at counts around those that
the kernel distinguishes, against the same cones taken a few at a time: the loss is a sum over cones,
and so is its gradient."""
import numpy as np
import pytest

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu

COEF = ((1.0, 0.01, 1.0), (0.5, 0.02, -1.0))


def _gradient(sc, weight, steps, every):
    M = sc.n_cones
    with B.Simulation(sc) as sim:
        sim.adjoint(steps, np.arange(M) % 30, weight, every)
        return np.concatenate(sim.adjoint_backward())


@pytest.mark.parametrize("n,cones,species,gathered", [
    ((112, 22), 128, 1, False), ((112, 22), 129, 1, False), ((113, 23), 200, 2, False),
    ((64, 48), 640, 1, False), ((64, 48), 641, 2, False), ((61, 47), 3000, 1, False),
    ((400, 301), 129, 1, True), ((400, 300), 700, 2, True), ((301, 200), 1200, 1, True),
])
def test_crowds(n, cones, species, gathered):
    print(f"[gpu] {n} {cones} cones {species} species {gathered}", flush=True)
    sc = S.make_scenario("crowd", 2, n, 1.0, 0.15, COEF[:species], 5, (0.5, 2.0), cones, 30, seed=6)
    sc.turn_gain = 0.2   # so that turns are seldom capped, and most samples have an adjoint
    if gathered:   # around one place
        rng = np.random.default_rng(4)
        sc.cone_pos = (np.array(n) * 0.5 + rng.uniform(-6.0, 6.0, (cones, 2))).astype(
            np.float32).astype(np.float64)
        for spc in sc.species:   # where the cue reaches them
            at = rng.integers(-4, 5, (len(spc.source_q), 2)) + np.array(n) // 2
            spc.source_cell = (at[:, 1] * n[0] + at[:, 0]).astype(np.int32)
    weight = np.linspace(0.5, 1.5, cones).astype(np.float32)
    whole = _gradient(sc, weight, 21, 13)
    assert np.all(whole == _gradient(sc, weight, 21, 13))
    # cones of weight 0 have no adjoint: at most 100 of the rest in any tile
    parts, size = [], np.zeros_like(whole)
    for lo in range(0, cones, 100):
        w = np.zeros_like(weight)
        w[lo:lo + 100] = weight[lo:lo + 100]
        parts.append(_gradient(sc, w, 21, 13))
        size += np.abs(parts[-1])
    # The field adjoint is FP32 (2^-24 per operation): each cell's is rounded 5 times per step (the
    # samples' sum, the stencil), the sums over cells are FP64; both sides, 21 steps of growth.
    tol = 2 * 21 * 5 * 2.0 ** -24
    err = np.abs(np.sum(parts, axis=0) - whole)
    assert np.all(size > 0)
    scale = np.maximum(size, 1e-3 * size.max())
    print(f"[gpu] largest error {np.max(err / scale):.2e} of its terms, bound {tol:.2e}", flush=True)
    assert np.all(err <= tol * scale)
