"""CPU check of how many maps a launch of the map mode builds at once, for any
number of maps that the interface takes (tests/host/map_builders_check.cpp)."""
import os
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists(f"{ROCM}/include/hip/hip_runtime.h"),
                    reason="needs g++ and the HIP headers")
def test_map_builders():
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "map_builders_check")
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", "-o", exe,
                               os.path.join(ROOT, "tests", "host", "map_builders_check.cpp")])
        out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
        assert out.returncode == 0 and out.stdout == "OK\n", out.stdout + out.stderr
