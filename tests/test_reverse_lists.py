"""The room for the lists of cones that touch a reverse tile, against the tiles that tips of wide
grids do touch, with their FP32 rounding (host code, on the CPU)."""
import os
import subprocess

import pytest

from paper_1405_3331_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1405_3331_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_capacity_counts_rounding(tmp_path):
    if not os.path.exists(B.LIBRARY):
        from paper_1405_3331_amd import build
        build.build()
    exe = str(tmp_path / "list_capacity_driver")
    subprocess.run([HIPCC, "-O2", "-std=c++17", "-ffp-contract=off", "--cuda-host-only", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), "-x", "hip",
                    os.path.join(HERE, "device_math", "list_capacity_driver.cpp"), "-x", "none",
                    B.LIBRARY, f"-Wl,-rpath,{os.path.dirname(B.LIBRARY)}", "-o", exe],
                   check=True, capture_output=True, timeout=300)
    # tiles of 112 x 22 cells, a halo of 8
    run = subprocess.run([exe, "112", "22", "8"], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout
    most, checked = (int(v) for v in run.stdout.split())
    assert most >= 3 and checked > 10 ** 5
