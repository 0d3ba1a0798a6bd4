"""Temporally blocked steps captured in a caller's graph: replayed, they are the steps that follow,
whatever the number of launches and replays, with reads, writes and eager steps between replays."""
import numpy as np
import pytest
import torch

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu

COEF = ((1.0, 0.01, 1.0), (0.5, 0.02, -1.0))


def _state(sim, species):
    cones = sim.cones()
    return [sim.field(s) for s in range(species)] + [cones[k] for k in sorted(cones)] + [sim.mass()]


@pytest.mark.parametrize("captured,block_steps,species", [
    (16, 0, 1), (24, 0, 2), (8, 8, 1), (16, 8, 2), (37, 12, 1), (5, 0, 1),
])
@pytest.mark.parametrize("between", ["nothing", "reads", "eager", "writes"])
def test_replays_follow_on(captured, block_steps, species, between):
    print(f"[gpu] {captured} steps at depth {block_steps}, {species} species, {between}", flush=True)
    sc = S.make_scenario("capture", 2, (200, 150), 1.0, 0.15, COEF[:species], 5, (0.5, 2.0), 900, 20,
                         seed=3)
    stream = torch.cuda.Stream()
    with B.Simulation(sc, stream=stream, block_steps=block_steps) as sim, \
            B.Simulation(sc, block_steps=1) as ref:
        sim.step(3).synchronize()
        ref.step(3)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sim.step(captured)
        for replay in range(5):
            with torch.cuda.stream(stream):
                graph.replay()
            ref.step(captured)
            if between == "reads" or replay == 4:
                for got, want in zip(_state(sim, species), _state(ref, species)):
                    np.testing.assert_array_equal(got, want)
            elif between == "eager":
                sim.step(7)
                ref.step(7)
            elif between == "writes":
                field = sim.field()
                np.testing.assert_array_equal(field, ref.field())
                sim.write(B.FIELD, field * 0.5)
                ref.write(B.FIELD, field * 0.5)
                pos = sim.cones()["pos"][::-1].copy()
                np.testing.assert_array_equal(pos[::-1], ref.cones()["pos"])
                for one in (sim, ref):
                    one.write(B.CONE_POS, pos)
                    one.step(1)   # (buckets the cones: a graph's launches do not)
