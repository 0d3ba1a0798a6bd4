"""The library's device memory pool on the CPU, over a stand-in for the runtime: what it keeps is
bounded by the device's memory, is given back when an allocation fails and on request, and is safe
with several threads (also under the thread and address sanitizers)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1405_3331_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(not os.path.isdir(os.path.join(ROCM, "include", "hip")),
                    reason="no HIP headers")
@pytest.mark.parametrize("sanitizer", ["", "thread", "address,undefined"])
def test_pool(tmp_path, sanitizer):
    exe = str(tmp_path / "pool_driver")
    san = [f"-fsanitize={sanitizer}"] if sanitizer else []
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", *san, "-D__HIP_PLATFORM_AMD__", "-I", CSRC,
                    "-I", os.path.join(ROCM, "include"), "-x", "c++",
                    os.path.join(CSRC, "memory.hip"),
                    os.path.join(HERE, "device_math", "pool_driver.cpp"), "-pthread", "-o", exe],
                   check=True, capture_output=True, timeout=300)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120,
                         env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert run.stdout.strip() == "ok", run.stdout + run.stderr[-2000:]
