"""Failing allocations and byte caps at the C entry points, on the CPU: tests/c_entry_check.cpp
builds the host code against a stand-in for the HIP runtime."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2507_15121_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_c_entry_points_when_allocations_fail(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path / "c_entry_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fopenmp", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"),
                        "-I" + CSRC, "-I" + os.path.join(ROOT, "include"), os.path.join(HERE, "c_entry_check.cpp"),
                        os.path.join(CSRC, "api.cpp"), os.path.join(CSRC, "layout.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300, env=dict(os.environ, OMP_NUM_THREADS="2"))
    assert r.returncode == 0 and "0 failures" in r.stdout, (r.stdout[-3000:] + r.stderr[-2000:])
