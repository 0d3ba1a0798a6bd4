"""The reverse field steps by tiles (112 x 22 cores, eight steps per launch) against the
oracle's reverse sweep, where a tile or a launch can go wrong: grids one cell past a tile,
odd row lengths, tiles away from every wall, launches of one to eight steps, tiles crowded
with more cones than are held in LDS (128), more sources than threads (512), and cones that
cross several tiles during a launch.  Each component within the bounds of the other gradient
tests (test_gpu_adjoint.py)."""
import math

import numpy as np
import pytest

from paper_1405_3331_amd import scenarios
from test_gpu_adjoint import _built, _compare  # noqa: F401  (the fixture builds the oracle)

pytestmark = pytest.mark.gpu


def _case(n, cones, seed, species=1, sources=4, step_len=0.5, targets=12):
    coef = ((1.0, 0.01, 1.0), (0.6, 0.02, -1.0))[:species]
    return scenarios.make_scenario("reverse tiles", 2, n, 1.0, 0.2, coef, sources, (2.0, 8.0),
                                   cones, targets, 1.0, step_len, 10.0, math.pi / 30.0, 0.1,
                                   seed=seed)


@pytest.mark.parametrize("n,species", [((112, 22), 1), ((113, 23), 2), ((225, 45), 1),
                                       ((360, 90), 2), ((361, 89), 1)])
def test_tile_edges(n, species):
    _compare(_case(n, 60, 31, species), 40, 20)


@pytest.mark.parametrize("steps,every", [(1, 1), (7, 7), (8, 8), (9, 9), (17, 16)])
def test_launch_lengths(steps, every):
    _compare(_case((130, 60), 40, 32), steps, every)


def test_crowded_tile():
    _compare(_case((100, 40), 420, 33, species=2), 24, 12)


def test_more_sources_than_threads_in_a_tile():
    _compare(_case((110, 21), 40, 34, sources=700), 20, 10)


def test_cones_crossing_tiles():
    _compare(_case((400, 120), 60, 35, step_len=9.0), 16, 16)
