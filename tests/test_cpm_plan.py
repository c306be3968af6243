"""The launch plan of the matrix-core nnCP kernel gives every unit of its two products to exactly one
wave, for all shapes and thread counts that the kernel takes: cpm_plan_check.cpp with a host compiler."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1909_07570_amd", "csrc")


def test_every_unit_comes_up_once(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "cpm_plan_check")
    b = subprocess.run([cxx, "-std=c++17", "-O2", "-I" + CSRC, "-o", exe, os.path.join(HERE, "cpm_plan_check.cpp")],
                       capture_output=True, text=True)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
