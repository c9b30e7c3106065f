"""The register transforms of the line kernel, the tile pair stage and the inverse (dftn.hpp) compiled for the host:
every length they are used at, in float64 against plain sums and in float32 for errors with a sign."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# what dftn.hpp needs of the HIP headers
STUB = """#pragma once
#include <cmath>
#include <cstdint>
#define __device__
#define __forceinline__ inline
struct float2 { float x, y; };
struct double2 { double x, y; };
inline float2 make_float2(float x, float y) { return {x, y}; }
inline double2 make_double2(double x, double y) { return {x, y}; }
"""


def test_register_transforms_on_the_host(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(STUB)
    exe = str(tmp_path / "register_transforms")
    subprocess.run([cxx, "-O1", "-std=c++17", "-ffp-contract=off", "-I", str(tmp_path),
                    "-I", os.path.join(ROOT, "paper_0909_0001_amd", "csrc"),
                    os.path.join(ROOT, "tests", "register_transforms_driver.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
