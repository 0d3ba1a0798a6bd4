"""Launches over the widest and thinnest grids that are accepted stay within what the runtime takes
(host code of the library, on the CPU)."""
import os
import subprocess

import pytest

from paper_1405_3331_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1405_3331_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_launch_sizes(tmp_path):
    if not os.path.exists(B.LIBRARY):
        from paper_1405_3331_amd import build
        build.build()
    exe = str(tmp_path / "launch_sizes_driver")
    subprocess.run([HIPCC, "-O2", "-std=c++17", "--cuda-host-only", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), "-x", "hip",
                    os.path.join(HERE, "device_math", "launch_sizes_driver.cpp"), "-x", "none",
                    B.LIBRARY, f"-Wl,-rpath,{os.path.dirname(B.LIBRARY)}", "-o", exe],
                   check=True, capture_output=True, timeout=300)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.stdout.strip() == "ok", run.stdout
