"""sim_release_memory: what released objects left is free for other allocators again, while objects
live and after, and what lives goes on."""
import numpy as np
import pytest
import torch

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_release():
    sc = S.make_scenario("release", 2, (150, 90), 1.0, 0.15, ((1.0, 0.01, 1.0),), 6, (0.5, 2.0), 300,
                         20, seed=3)
    big = S.make_scenario("release", 2, (2048, 2048), 1.0, 0.15, ((1.0, 0.01, 1.0),), 6, (0.5, 2.0),
                          20000, 20, seed=3)
    B.Simulation(sc).close()
    B.sim_release_memory()
    with B.Simulation(sc) as sim:
        sim.step(20)
        before = _free()
        with B.Simulation(big) as other:
            other.adjoint(20, np.arange(20000) % 20, np.ones(20000), 10)   # 0.4 GB of field states
            other.adjoint_backward()
        assert before - _free() > 1 << 28
        B.sim_release_memory()
        assert before - _free() <= 32 << 20
        sim.step(20)
        got = sim.field()
    with B.Simulation(sc, block_steps=1) as sim:
        sim.step(40)
        np.testing.assert_array_equal(got, sim.field())
    B.sim_release_memory()
    assert _free() >= before
