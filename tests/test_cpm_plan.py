"""The launch plan of the matrix-core nnCP kernel gives every unit of its two products to exactly one
wave, for all shapes and thread counts that the kernel takes: cpm_plan_check.cpp with a host compiler."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1909_07570_amd", "csrc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("plan") / "cpm_plan_check")
    b = subprocess.run([cxx, "-std=c++17", "-O2", "-I" + CSRC, "-o", exe, os.path.join(HERE, "cpm_plan_check.cpp")],
                       capture_output=True, text=True)
    assert b.returncode == 0, b.stderr
    return exe


def test_every_unit_comes_up_once(exe):
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout


# modes, rank, threads and whether the matrix-core kernel takes the fit: either side of each line
@pytest.mark.parametrize("dims,rank,threads,mm", [
    ((40, 40, 40), 3, 1024, 0), ((33, 33, 33), 8, 1024, 0), ((21, 38, 61), 10, 1024, 0), ((21, 38, 61), 16, 1024, 1),
    ((20, 20, 20), 6, 512, 1), ((20, 20, 20), 6, 128, 0), ((20, 20, 20), 10, 1024, 1), ((24, 24, 24), 16, 1024, 1),
    ((9, 8, 8), 17, 512, 0), ((9, 8, 8), 16, 512, 1), ((9, 8, 8), 23, 512, 1), ((9, 10, 16), 20, 512, 1),
    ((2, 1, 51, 39), 8, 512, 0), ((7, 2, 53, 38), 3, 1024, 0), ((4, 8, 12, 16), 10, 1024, 1), ((8, 4, 64, 32), 8, 1024, 1),
    ((16, 16, 16, 16), 8, 1024, 1), ((8, 8, 8, 8, 8), 16, 1024, 1), ((2, 3, 4, 12, 12), 1, 256, 1)])
def test_route(exe, dims, rank, threads, mm):
    r = subprocess.run([exe, str(rank), str(threads)] + [str(n) for n in dims], capture_output=True, text=True)
    assert r.returncode == 0 and int(r.stdout) == mm
