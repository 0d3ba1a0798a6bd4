"""The tiled launch's own bookkeeping against the per-step path, bit for bit: tiles with more
sources and targets than their fixed-stride heads hold (64), crowded tiles whose further parts
are listed while the cones are bucketed, and reads between launches, which leave the buckets
in place, followed by writes, which do not."""
import numpy as np
import pytest

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu


def _case(cones, sources, targets, seed, n=(128, 96), crowd=False):
    sc = S.make_scenario("tile parts", 2, n, 1.0, 0.2, ((1.0, 0.01, 1.0),), sources, (0.5, 2.0),
                         cones, targets, seed=seed)
    if crowd:   # every cone starts inside one tile's core
        sc.cone_pos = np.asarray(sc.cone_pos * 0.05 + 40.0, np.float32).astype(np.float64)
    return sc


def _state(sim):
    return dict(sim.cones(), field=sim.field())


def _same(a, b, what):
    for k in a:
        assert np.array_equal(a[k], b[k]), (what, k)


@pytest.mark.parametrize("cones,sources,targets,crowd", [
    (40, 63, 64, False), (40, 64, 65, False), (200, 200, 300, False), (193, 4, 8, True),
    (512, 4, 8, True), (513, 4, 8, True), (2100, 70, 70, True)])
def test_heads_and_parts(cones, sources, targets, crowd):
    sc = _case(cones, sources, targets, 5, crowd=crowd)
    with B.Simulation(sc, block_steps=8) as tiled, B.Simulation(sc, block_steps=1) as plain:
        for steps in (8, 1, 16, 3):
            tiled.step(steps)
            plain.step(steps)
        _same(_state(tiled), _state(plain), (cones, sources, targets))


def test_read_leaves_buckets_and_write_replaces_them():
    sc = _case(700, 6, 20, 6)
    with B.Simulation(sc, block_steps=8) as tiled, B.Simulation(sc, block_steps=1) as plain:
        for sim in (tiled, plain):
            sim.step(10)
            sim.counts()                       # read, step on from the buckets
            sim.step(5)
            c = sim.cones()
            sim.cones()                        # nothing stepped in between
            sim.write(B.CONE_POS, c["pos"][::-1].copy())
            sim.write(B.CONE_STATUS, c["status"][::-1].copy())
            assert np.array_equal(sim.cones()["pos"], c["pos"][::-1])
            sim.step(11)
        _same(_state(tiled), _state(plain), "after a write")


def test_batch_read_between_launches():
    scs = [_case(900, 8, 30, 7 + i, n=(90 + 40 * i, 70), crowd=i == 1) for i in range(3)]
    with B.Batch(scs, graph_launches=2, block_steps=8) as bt:
        for steps in (16, 5, 24):
            bt.step(steps)
            bt.cones(1)
        for i, sc in enumerate(scs):
            with B.Simulation(sc, block_steps=1) as one:
                one.step(45)
                assert np.array_equal(bt.field(i), one.field()), i
                _same(bt.cones(i), one.cones(), i)


def test_volume_read_between_steps():
    sc = S.make_scenario("volume reads", 3, (24, 20, 18), 1.0, 0.15,
                         ((1.0, 0.01, 1.0), (0.5, 0.02, -1.0)), 6, (0.5, 2.0), 400, 30, seed=8)
    with B.Simulation(sc) as read, B.Simulation(sc) as straight:
        for steps in (3, 40, 7):
            read.step(steps)
            read.cones()
        straight.step(50)
        _same(_state(read), _state(straight), "reads")
        for sim in (read, straight):
            sim.write(B.CONE_DIR, -sim.cones()["dir"])
            sim.step(5)
        _same(_state(read), _state(straight), "after a write")
