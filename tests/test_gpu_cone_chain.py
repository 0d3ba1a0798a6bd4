"""The cones' reverse chain beside the reverse field steps of the segment after (a run whose record
fits) against the chain in launches of its own, segment by segment (a run that is re-run from its
checkpoints): the same states and the same order of every cone's steps.  Segments shorter than,
equal to and longer than a launch's eight steps, a last segment with fewer launches than the one
before it, and a single segment."""
import numpy as np
import pytest

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu

COEF = ((1.0, 0.01, 1.0), (0.5, 0.02, -1.0))


@pytest.mark.parametrize("species", [1, 2])
@pytest.mark.parametrize("steps,every,cones", [
    (10, 100, 70), (17, 8, 513), (40, 7, 64), (41, 20, 700), (65, 64, 1), (66, 33, 1200),
])
def test_chain_beside_the_fields(steps, every, cones, species):
    print(f"[gpu] {steps} steps, every {every}, {cones} cones, {species} species", flush=True)
    sc = S.make_scenario("chain", 2, (151, 120), 1.0, 0.15, COEF[:species], 8, (0.5, 2.0), cones,
                         30, seed=12)
    out = []
    for limit in (0, 1):   # a byte holds no record: every segment is re-run
        with B.Simulation(sc) as sim:
            sim.set_tape_limit(limit)
            loss = sim.adjoint(steps, np.arange(cones) % 30, np.linspace(0.5, 1.5, cones), every)
            out.append([np.array(loss)] + [np.array(v) for v in sim.adjoint_backward()])
    for a, b in zip(*out):
        # FP64 sums over tiles: their number and order are the same either way
        np.testing.assert_allclose(b, a, rtol=1e-13, atol=0.0)
