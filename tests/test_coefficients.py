"""The collision's coefficients conserve mass and momentum by their sums,
exactly in each precision: a sum that misses 1 by a rounding acts the same way
at every step and grows with the run."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_coefficient_sums_close_exactly(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path / "coef_check")
    subprocess.run([gxx, "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
                    os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_0707_2437_amd", "csrc"),
                    os.path.join(ROOT, "tests", "coef_check.cpp"), "-o", exe, "-L/opt/rocm/lib", "-lamdhip64"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "coefficients ok", r.stdout + r.stderr
