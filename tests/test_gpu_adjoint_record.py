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


def _limits(sc, steps):
    """Tape limits that hold everything, the field states and 16 bytes per cone step, nothing."""
    fields = 4 * (steps + 1) * len(sc.species) * sc.n_cells
    alone = fields + 16 * steps * sc.n_cones
    whole = fields + (80 if len(sc.species) == 1 else 112) * steps * sc.n_cones
    return {"all": whole + 1, "all but a byte": whole, "fields": alone + 1, "fields but a byte": alone,
            "none": 1}


@pytest.mark.parametrize("species", [1, 2])
@pytest.mark.parametrize("steps,every,cones,block_steps", [
    (10, 100, 70, 0), (70, 7, 513, 0), (90, 4, 64, 1), (41, 20, 700, 0), (33, 1, 40, 0),
    (66, 33, 1200, 5), (130, 11, 3, 0),
])
def test_every_way_to_record(steps, every, cones, species, block_steps):
    """Everything recorded, the field states alone (the cones re-run, windows of several segments
    that do not divide the run), nothing, or nothing and then room for the whole run: the same loss
    and gradient, bit for bit."""
    print(f"[gpu] {steps} steps, every {every}, {cones} cones, {species} species", flush=True)
    sc = _case(species, cones, seed=17)
    assign, weight = np.arange(cones) % 20, np.linspace(0.5, 1.5, cones)
    want = None
    limits = _limits(sc, steps)
    for name, after in [(k, None) for k in limits] + [("none", "all"), ("fields", "all"),
                                                      ("all", "none"), ("none", "fields")]:
        with B.Simulation(sc, block_steps=block_steps) as sim:
            sim.set_tape_limit(limits[name])
            out = [np.array(sim.adjoint(steps, assign, weight, every))]
            if after:
                sim.set_tape_limit(limits[after])
            for _ in range(2):
                got = out + [np.array(v) for v in sim.adjoint_backward()]
                want = want or got
                for g, v in zip(got, want):
                    np.testing.assert_array_equal(g, v, err_msg=f"{name}, {after}")
