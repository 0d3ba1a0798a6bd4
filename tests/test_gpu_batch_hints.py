"""Batches whose members ask for tile heights and leave the depth to the library: made, and every
member equal bit for bit to the same simulation at one step per launch."""
import copy

import numpy as np
import pytest

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hints", [(64, 0), (64, 96), (60, 110), (44, 0, 300), (10, 0)])
def test_hinted_members(hints):
    print(f"[gpu] heights {hints}", flush=True)
    sizes = [(150, 150), (200, 333), (90, 80)]
    scs = [S.make_scenario("hints", 2, sizes[i], 1.0, 0.2, ((1.0, 0.01, 1.0),), 5, (0.5, 2.0), 300,
                           12, seed=20 + i, sim_index=i) for i in range(len(hints))]
    for sc, hint in zip(scs, hints):
        sc.tile = (0, hint)
    with B.Batch([copy.copy(sc) for sc in scs], graph_launches=2) as bt:
        bt.step(53)
        for i, sc in enumerate(scs):
            if hints[i] >= 44:
                assert bt.tiling(i)["height"] == hints[i]
            with B.Simulation(sc, block_steps=1) as one:
                one.step(53)
                np.testing.assert_array_equal(bt.field(i), one.field())
                want, got = one.cones(), bt.cones(i)
                for k in want:
                    np.testing.assert_array_equal(got[k], want[k])
