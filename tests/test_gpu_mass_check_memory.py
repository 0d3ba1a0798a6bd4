"""A mass check is set on a handle without a call that a stream capture forbids (its buffers were
made with the handle), and works afterwards."""
import numpy as np
import pytest
import torch

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n", [(2, (50, 40)), (3, (12, 10, 9))])
def test_set_during_a_capture(dim, n):
    sc = S.make_scenario("mass", dim, n, 1.0, 0.1, ((1.0, 0.01, 1.0),), 3, (0.5, 2.0), 20, 5)
    x = torch.zeros(1000, device="cuda")
    with B.Simulation(sc) as sim:
        sim.step(3).synchronize()
        stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="global"):
            x += 1.0
            sim.set_mass_check(4)
        graph.replay()
        graph.replay()
        torch.cuda.synchronize()
        assert x.eq(2.0).all()
        sim.step(9).synchronize()
        bad = sim.field()
        want = float(bad.astype(np.float64).sum())
        assert abs(sim.mass()[0] - want) <= 1e-9 * abs(want)
        bad.flat[7] = np.inf
        sim.write(B.FIELD, bad)
        sim.step(8)
        with pytest.raises(B.SimError) as e:
            sim.synchronize()
        assert e.value.status == B.SIM_ENONFINITE


def test_many_handles():
    """More handles than a page holds words, some made after others went."""
    sc = S.make_scenario("mass", 2, (16, 12), 1.0, 0.1, ((1.0, 0.01, 1.0),), 3, (0.5, 2.0), 4, 2)
    sims = [B.Simulation(sc) for _ in range(70)]
    bad = np.full(sc.shape, np.nan, dtype=np.float32)
    for k, sim in enumerate(sims):
        sim.set_mass_check(2)
        if k % 3 == 0:
            sim.write(B.FIELD, bad)
        sim.step(2)
    for k, sim in enumerate(sims):
        if k % 3 == 0:
            with pytest.raises(B.SimError):
                sim.synchronize()
            sim.close()
        else:
            sim.synchronize()
    for sim in [B.Simulation(sc) for _ in range(30)] + [s for k, s in enumerate(sims) if k % 3]:
        sim.set_mass_check(2).step(2).synchronize()
        sim.close()
