"""What a gradient's record holds when the run behind it did not go to its end, or when the state was
written after it."""
import numpy as np
import pytest

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu


def _case(species=1, cones=200, seed=5):
    coef = ((1.0, 0.01, 1.0), (0.5, 0.02, -1.0))
    return S.make_scenario("record", 2, (140, 100), 1.0, 0.15, coef[:species], 6, (0.5, 2.0), cones,
                           20, seed=seed)


@pytest.mark.parametrize("block_steps", [0, 1])
def test_a_failed_run_leaves_no_record(block_steps):
    """A mass check that found a non-finite total stops the run at its first segment.  Stepping on
    from a mended state to the run's last step does not make it one to differentiate."""
    sc = _case()
    M = sc.n_cones
    assign, weight = np.arange(M) % 20, np.ones(M)
    with B.Simulation(sc, block_steps=block_steps) as sim:
        sim.adjoint(40, assign, weight, 10)          # an earlier record, which the call replaces
        sim.set_mass_check(4)
        good = sim.field()
        bad = good.copy()
        bad[3, 5] = np.nan
        sim.write(B.FIELD, bad)
        sim.step(4)
        with pytest.raises(B.SimError) as e:
            sim.synchronize()
        assert e.value.status == B.SIM_ENONFINITE
        with pytest.raises(B.SimError) as e:
            sim.adjoint(40, assign, weight, 10)
        assert e.value.status == B.SIM_ENONFINITE
        sim.write(B.FIELD, good)
        assert np.isfinite(sim.mass()).all()
        sim.step(40)
        with pytest.raises(B.SimError) as e:
            sim.adjoint_backward()
        assert e.value.status == B.SIM_ESTATE
        sim.adjoint(40, assign, weight, 10)          # and the next one stands
        assert all(np.isfinite(v).all() for v in sim.adjoint_backward())


@pytest.mark.parametrize("species,limit", [(1, 0), (1, 1), (2, 0), (2, 1)])
def test_states_written_after_the_run(species, limit):
    """The record holds no steps past a cone's stop: a status written after the run that says the
    cone went on changes nothing, and one that says it stopped earlier leaves its later steps out
   ."""
    sc = _case(species, cones=400, seed=8)
    sc.contact_radius = 2.0
    M = sc.n_cones
    assign, weight = np.arange(M) % 20, np.linspace(0.5, 1.5, M)
    with B.Simulation(sc) as sim:
        sim.set_tape_limit(limit)
        sim.adjoint(60, assign, weight, 17)
        want = [np.array(v) for v in sim.adjoint_backward()]
        c = sim.cones()
        stopped = c["status"] != B.ACTIVE
        assert 10 < stopped.sum() < M
        sim.write(B.CONE_STATUS, np.zeros(M, dtype=np.int32))
        for got, v in zip(sim.adjoint_backward(), want):
            np.testing.assert_array_equal(got, v)
        sim.write(B.CONE_STATUS, c["status"])
        sim.write(B.CONE_EVENT_STEP, np.full(M, 10 ** 6, dtype=np.int32))
        for got, v in zip(sim.adjoint_backward(), want):
            np.testing.assert_array_equal(got, v)
        # every cone stopped before the run's first step: nothing takes part
        sim.write(B.CONE_STATUS, np.full(M, B.EXITED, dtype=np.int32))
        sim.write(B.CONE_EVENT_STEP, np.zeros(M, dtype=np.int32))
        assert not any(np.any(v) for v in sim.adjoint_backward())
        sim.write(B.CONE_STATUS, c["status"])
        sim.write(B.CONE_EVENT_STEP, c["event_step"])
        for got, v in zip(sim.adjoint_backward(), want):
            np.testing.assert_array_equal(got, v)
