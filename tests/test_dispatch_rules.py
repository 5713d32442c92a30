"""The rules that choose between kernels by sizes (host code, no GPU): compiled
from the library's internal header and checked on both sides of their lines."""

import os
import shutil
import subprocess

import pytest

from paper_1904_00962_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_rules_on_both_sides_of_their_lines(tmp_path):
    gxx = shutil.which("g++")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if gxx is None or not os.path.exists(os.path.join(rocm, "include", "hip")):
        pytest.skip("needs g++ and the HIP headers")
    exe = tmp_path / "rules"
    r = subprocess.run([gxx, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", build.INCLUDE,
                        "-I", build.CSRC, "-I", os.path.join(rocm, "include"),
                        os.path.join(HERE, "dispatch_rules.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
