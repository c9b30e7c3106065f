"""Schedules of the general (line) kernel on the CPU: the planner's tables, strides, splits and divisions executed
in float64 with bounds checks by tests/lines_schedule_driver.cpp, against plain zero-padded DFTs, for axes of every
length up to 64 whose prime factors have a register transform, mixed-size grids of one to eight axes, grids that are
split among work-groups, and beam-space grids (unpadded innermost axes); and the inverse's groups for the same
grids, one to 40 channels, with and without values behind the last axis, against plain inverse sums."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_0909_0001_amd", "csrc")


def smooth(v):
    for p in (2, 3, 5, 7, 11, 13):
        while v % p == 0:
            v //= p
    return v == 1


GRIDS = [f"{n}" for n in range(1, 65) if smooth(n)] + ["128", "240", "512"]
GRIDS += [f"{n} {k}" for n, k in [(2, 3), (3, 5), (16, 16), (6, 10), (8, 8), (9, 15), (20, 24), (7, 13), (32, 16), (40, 39)]]
GRIDS += ["64 48", "96 32", "128 24", "26 64", "19 4", "34 2"]  # split along axis 0
GRIDS += ["5 3 3 3 3 3", "2 2 16 16", "3 3 3 3 5 3", "4 4 4 4", "4 4 4 4 4", "8 8 4 4", "6 5 4 3 2", "2 2 2 2 2 2", "2 2 2 2 2 2 2 2", "12 3 12"]
# short axes two by two: every pair of lengths that is one pass, alone and behind another axis
GRIDS += [f"{a} {b}" for a in range(2, 9) for b in range(2, a + 1) if a * b <= 16] + ["2 8 2 8", "3 4 7 2", "5 3 16", "11 3 3"]
GRIDS += ["4 4 8 8 b2", "2 3 3 3 4 4 b2", "3 3 5 5 b2", "4 8 b1", "6 5 9 10 b2", "4 4 16 12 b2", "7 7 b1"]
# prime factors without a register transform; a grid that axis 0 cannot divide far enough
NOT_PLANNED = ["17", "4 19", "3 34", "5 5 23 b1", "2 2 16 16 16"]


def test_line_schedules_against_plain_dfts(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "lines_schedule")
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", CSRC, os.path.join(ROOT, "tests", "lines_schedule_driver.cpp"),
                    os.path.join(CSRC, "lines_plan.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], input="\n".join(GRIDS) + "\n", capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert f"schedules checked: {2 * len(GRIDS)}" in r.stdout and "not planned: 0" in r.stdout, r.stdout
    r = subprocess.run([exe], input="\n".join(NOT_PLANNED) + "\n", capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "schedules checked: 0" in r.stdout, r.stdout + r.stderr
