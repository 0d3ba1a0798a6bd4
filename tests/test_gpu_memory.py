"""Device memory reused between the library's objects: results do not depend on what a block
held before, several threads and streams may create, run and destroy objects at once, and what
is kept between objects is bounded."""
import threading

import numpy as np
import pytest
import torch

from paper_1405_3331_amd import binding as B
from paper_1405_3331_amd import scenarios as S

pytestmark = pytest.mark.gpu


def _case(seed, n=(150, 90), cones=300, dim=2):
    coef = ((1.0, 0.01, 1.0), (0.5, 0.02, -1.0))
    return S.make_scenario("memory", dim, n, 1.0, 0.15, coef, 6, (0.5, 2.0), cones, 20,
                           seed=seed)


def _run(sc, stream=None, gradient=True):
    with B.Simulation(sc, stream=stream) as sim:
        out = []
        if gradient:
            M = sc.n_cones
            out.append(sim.adjoint(30, np.arange(M) % 20, np.linspace(0.5, 1.5, M), 11))
            out += [np.array(v) for v in sim.adjoint_backward()]
        else:
            sim.step(30)
        owner = np.arange(sc.n_cones) % 7
        out += list(sim.connectivity(7, owner, np.arange(20) % 7))
        out.append(sim.bfs_levels(0, 7))
        out += [sim.mass(), sim.field(0), sim.field(1)] + list(sim.cones().values())
    return out


def _same(a, b):
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def test_results_do_not_depend_on_reused_memory():
    """The same objects made after others of nearly the same size have filled their memory."""
    first = _run(_case(1))
    volume = _run(_case(2, (30, 22, 18), dim=3), gradient=False)
    for seed in (3, 4):
        _run(_case(seed, (149, 92), 310))
        _run(_case(seed, (31, 22, 18), 290, dim=3), gradient=False)
    _same(_run(_case(1)), first)
    _same(_run(_case(2, (30, 22, 18), dim=3), gradient=False), volume)


def test_threads_and_streams():
    cases = [_case(10 + k, (120 + 8 * k, 70), 200 + k) for k in range(4)]
    want = [_run(sc) for sc in cases]
    got = [None] * len(cases)
    errors = []

    def work(k):
        try:
            stream = torch.cuda.Stream()
            for _ in range(6):
                got[k] = _run(cases[k], stream=stream if k % 2 else None)
                _same(got[k], want[k])
        except BaseException as e:   # noqa: BLE001  (reported by the main thread)
            errors.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_memory_between_objects_is_bounded():
    """Three simulations with a gigabyte of cone slots each leave at most a gigabyte behind."""
    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    _run(_case(5))   # the runtime's own allocations
    before = free()
    sims = []
    for k in range(3):
        sc = S.headline(seed=k)
        sc.tile = (2, 143)   # 480 tiles
        sims.append(B.Simulation(sc, block_steps=12))
    assert before - free() > 3 << 29
    for sim in sims:
        sim.step(12)
        sim.close()
    assert before - free() <= (1 << 30) + (64 << 20)
