"""Adjacency and levels at the edges of the sort's and the traversal's ranges: a tile of the sort
and one item more or less, as many tiles as a scatter adds up itself and one more, one and two
digits of keys, graphs for one launch and for a launch per level, long paths and a vertex that
owns every edge.  Whole numbers, equal to the oracle's."""
import numpy as np
import pytest

import oracle
from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _built(oracle_lib):
    return oracle_lib


CASES = [  # connections, neurons, kind
    (1, 1, "random"), (2047, 255, "random"), (2048, 256, "random"), (2049, 300, "random"),
    (65536, 4096, "random"), (65537, 16384, "random"), (140000, 32768, "random"),
    (140000, 32769, "random"), (262144, 3000, "random"), (262145, 3000, "random"),
    (3000, 3001, "path"), (70000, 20000, "star"),
]


@pytest.mark.parametrize("m,n,kind", CASES)
def test_adjacency_and_levels(m, n, kind):
    print(f"[gpu] {kind}: {m} cones, {n} neurons", flush=True)
    rng = np.random.default_rng(m + n)
    t = min(n, 4096) if kind == "random" else n
    sc = S.make_scenario("graph", 2, (48, 40), n_cones=m, n_targets=t, n_sources=1, seed=1)
    towner = rng.integers(0, n, t) if kind == "random" else np.arange(n)
    if kind == "random":
        owner, target = rng.integers(0, n, m), rng.integers(0, t, m)
        status = (rng.random(m) < 0.8).astype(np.int32)
        status[:1] = 1
    elif kind == "path":   # cone i joins neuron i to i + 1
        owner, target, status = np.arange(m), np.arange(1, m + 1), np.ones(m, np.int32)
    else:
        owner, target = np.full(m, 7), rng.integers(0, n, m)
        status = np.ones(m, np.int32)
    with B.Simulation(sc, block_steps=1) as sim:
        sim.write(B.CONE_STATUS, status)
        sim.write(B.CONE_TARGET, np.where(status == 1, target, -1).astype(np.int32))
        row, edges = sim.connectivity(n, owner, towner)
        row_ref, edges_ref = oracle.connectivity(n, status, target, owner, towner)
        np.testing.assert_array_equal(row, row_ref)
        np.testing.assert_array_equal(edges, edges_ref)
        for root in {0, int(owner[0]), n - 1}:
            np.testing.assert_array_equal(sim.bfs_levels(root, n),
                                          oracle.bfs_levels(row_ref, edges_ref, root))
