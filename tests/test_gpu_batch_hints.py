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


@pytest.mark.parametrize("n,step_len,depth,tile", [
    ((600, 420), 31.0, 0, (0, 0)), ((300, 300), 4.5, 16, (0, 30)), ((300, 300), 4.5, 16, (4, 30)),
    ((200, 150), 12.0, 0, (2, 0)),
])
def test_one_row_width(n, step_len, depth, tile):
    """Shapes that leave no core at the width asked for (or at two columns per lane): the batch
    takes the other width as a whole."""
    print(f"[gpu] {n} step {step_len} depth {depth} tile {tile}", flush=True)
    scs = [S.make_scenario("width", 2, n, 1.0, 0.2, ((1.0, 0.01, 1.0),), 5, (0.5, 2.0), 400, 12,
                           step_len=step_len, seed=30 + i, sim_index=i) for i in range(2)]
    for sc in scs:
        sc.tile = tile
    with B.Batch([copy.copy(sc) for sc in scs], block_steps=depth) as bt:
        assert bt.tiling(0)["cols_per_lane"] == bt.tiling(1)["cols_per_lane"]
        bt.step(29)
        for i, sc in enumerate(scs):
            with B.Simulation(sc, block_steps=1) as one:
                one.step(29)
                np.testing.assert_array_equal(bt.field(i), one.field())
                want, got = one.cones(), bt.cones(i)
                for k in want:
                    np.testing.assert_array_equal(got[k], want[k])
