"""What dugks_step enqueues (launches of one or two steps, captured graphs, the
buffer and the step index of each), on the CPU with stand-ins for the kernels and
the HIP calls (tests/host_schedule_driver.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1906_11036_amd", "csrc")
HIP_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")


def test_launch_schedule(tmp_path):
    if shutil.which("g++") is None or not os.path.isdir(os.path.join(HIP_INCLUDE, "hip")):
        pytest.skip("g++ or the HIP headers not found")
    exe = str(tmp_path / "driver")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-w", "-I", HIP_INCLUDE, "-I", CSRC,
                        "-I", os.path.join(ROOT, "include"), os.path.join(CSRC, "dugks_host.cpp"),
                        os.path.join(HERE, "host_schedule_driver.cpp"), "-o", exe, "-pthread"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "ok" in run.stdout, run.stderr[-3000:]
