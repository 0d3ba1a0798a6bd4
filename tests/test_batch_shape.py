"""The launch shape of a batch (host code of the library, on the CPU): one depth for all members,
whatever heights some of them ask for; a member's own height where it fits."""
import os
import subprocess

import pytest

from paper_1405_3331_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1405_3331_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")


@pytest.fixture(scope="module")
def shape(tmp_path_factory):
    if not os.path.exists(B.LIBRARY):
        from paper_1405_3331_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("shape") / "batch_shape_driver")
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--cuda-host-only", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), "-x", "hip",
                    os.path.join(HERE, "device_math", "batch_shape_driver.cpp"), "-x", "none",
                    B.LIBRARY, f"-Wl,-rpath,{os.path.dirname(B.LIBRARY)}", "-o", exe],
                   check=True, capture_output=True, timeout=300)

    def run(members, depth=0, cols=0, whole=False):
        """(planned depth, [(depth, height) of every member]); members: (nx, ny, species, step,
        cones, tile height).  whole: (misfit, width, depth, [(width, depth) of every member])."""
        args = [str(v) for m in members for v in m]
        out = subprocess.run([exe, str(depth), str(cols), *args], check=True, capture_output=True,
                             text=True, timeout=60).stdout.splitlines()
        v = [int(x) for x in out[1 if whole else 0].split()]
        if whole:
            return v[0], v[1], v[2], list(zip(v[3::2], v[4::2]))
        return v[0], list(zip(v[1::2], v[2::2]))
    return run


def _members(hints, step=0.5):
    sizes = [(150, 150), (200, 333)]
    return [(*sizes[i % 2], 1, step, 100, h) for i, h in enumerate(hints)]


@pytest.mark.parametrize("hints", [(64, 0), (0, 64), (64, 96), (60, 110), (44, 0), (44, 300),
                                   (138, 0, 64)])
def test_hinted_heights_share_a_depth(shape, hints):
    depth, plans = shape(_members(hints))
    assert depth >= 8
    for hint, (b, h) in zip(hints, plans):
        assert b == depth
        assert hint in (0, h)


@pytest.mark.parametrize("hint", [10, 5000])
def test_a_height_that_fits_no_depth_is_ignored(shape, hint):
    depth, plans = shape(_members((hint, 0)))
    free, free_plans = shape(_members((0, 0)))
    assert (depth, plans) == (free, free_plans)


def test_a_height_for_shallow_launches_only(shape):
    """Fits three steps and fewer: every member of a batch of such takes them, as alone."""
    depth, plans = shape(_members((30, 30)))
    assert depth == 0
    assert plans[0] == plans[1] and plans[0][1] == 30


def test_with_a_depth_asked_for(shape):
    depth, plans = shape(_members((80, 0)), depth=12)
    assert depth == 12
    assert plans[0] == (12, 80) and plans[1][0] == 12


@pytest.mark.parametrize("members,depth,cols,want", [
    ([(600, 600, 1, 31.0, 500, 0)] * 3, 0, 0, (4, 2)),      # no core at 128 columns
    ([(600, 600, 1, 31.0, 500, 0)] * 3, 0, 2, (4, 2)),
    ([(300, 300, 1, 4.5, 500, 30)] * 2, 16, 0, (2, 8)),     # a height that fits nowhere
    ([(300, 300, 1, 4.5, 500, 30)] * 2, 16, 4, (4, 9)),
    ([(300, 300, 1, 0.5, 500, 0), (80, 90, 1, 3.0, 5, 0)], 0, 0, (2, 8)),
    ([(300, 300, 2, 0.5, 500, 0)] * 2, 8, 4, (4, 8)),
])
def test_one_row_width(shape, members, depth, cols, want):
    misfit, width, steps, plans = shape(members, depth, cols, whole=True)
    assert misfit == -1 and (width, steps) == want
    assert all(p == want for p in plans)


def test_no_common_depth(shape):
    """A member that no launch as deep as the others' fits, at either row width."""
    members = [(600, 600, 1, 0.5, 500, 0), (600, 600, 1, 31.0, 500, 0)]
    assert shape(members, whole=True)[0] == 1
    assert shape([(600, 600, 1, 0.5, 500, 0), (600, 600, 1, 120.0, 500, 0)], whole=True)[0] == 1
