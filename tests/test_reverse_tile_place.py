"""Where the reverse sweep's tiles lie (tile_place) built for the host: every number of tiles to a
row, up to the widest grid that is accepted, at the first and the last tile of every row."""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1405_3331_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_every_row_of_tiles(tmp_path):
    # the core of a tile: 128 loaded columns less a halo of 8 on either side, 22 rows
    exe = str(tmp_path / "tile_place_driver")
    subprocess.run([HIPCC, "-O2", "-std=c++17", "-x", "hip", "--cuda-host-only", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"),
                    os.path.join(HERE, "device_math", "tile_place_driver.cpp"), "-o", exe],
                   check=True, capture_output=True, timeout=300)
    run = subprocess.run([exe, "112", "22"], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout
    assert int(re.match(r"(\d+) rows", run.stdout).group(1)) > 10 ** 7
