"""Copies of large arrays to host memory (csrc/host_copy.h: two pinned chunks
emptied by several threads), on the CPU with stand-ins for the HIP calls
(tests/host_copy_driver.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1906_11036_amd", "csrc")
HIP_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.isdir(os.path.join(HIP_INCLUDE, "hip")):
        pytest.skip("g++ or the HIP headers not found")
    exe = str(tmp_path_factory.mktemp("host_copy") / "driver")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-w", "-I", HIP_INCLUDE, "-I", CSRC,
                        os.path.join(HERE, "host_copy_driver.cpp"), "-o", exe, "-pthread"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.mark.parametrize("case", ["values", "idle", "devices", "direct"])
def test_host_copy(driver, case):
    r = subprocess.run([driver, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
