"""CPU-only: the host side of the library when host memory runs out (tests/host/build_without_memory.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2504_13989_amd", "csrc")


def test_building_a_handle_without_memory(tmp_path):
    gxx = shutil.which("g++")
    if not gxx or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(tmp_path / "build_without_memory")
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "host", "build_without_memory.cpp"), os.path.join(CSRC, "rotq_api.cpp"),
                    os.path.join(CSRC, "hadamard.cpp"), "-Wl,--unresolved-symbols=ignore-all", "-o", exe],
                   check=True, capture_output=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and run.stdout.strip() == "ok", run.stdout
