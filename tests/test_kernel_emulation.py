"""The single-pass kernels on the CPU: their own source, compiled for the host
over an emulated workgroup whose waves run as far ahead of each other as the
barriers allow (kernel_emulation.h). Layers with ragged ends that follow one
another on a workgroup must come out bit for bit as in a plan of one round,
whichever wave runs ahead: what one wave keeps in LDS for its writes, another
wave that is already on the next tile must not overwrite."""

import os
import shutil
import subprocess

import pytest

from paper_1904_00962_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def output(tmp_path_factory):
    tmp_path = tmp_path_factory.mktemp("emulation")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    clang = shutil.which("amdclang++") or os.path.join(rocm, "llvm", "bin", "clang++")
    if not os.path.exists(clang):
        pytest.skip("no clang++ (the kernel source uses its vector extension)")
    # the kernels' own include of the HIP device runtime finds an empty file
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text("")
    exe = tmp_path / "emulation"
    r = subprocess.run([clang, "-std=c++17", "-O1", "-ffp-contract=off", "-w", "-pthread",
                        "-I", str(tmp_path), "-I", build.INCLUDE, "-I", build.CSRC,
                        "-I", os.path.join(rocm, "include"),
                        os.path.join(HERE, "kernel_emulation.cpp"), "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    return r.stdout + r.stderr


def test_no_wave_overtakes_another(output):
    assert "all layers agree" in output, output[-2000:]


def test_an_eager_wait_gives_up_no_sooner(output):
    """A give-up counts polls, and an eager wait's are shorter: it gets more of
    them, so that a layer whose tiles are late on a busy device is waited for as
    long in a plan of one round as in any other."""
    assert "all waits are as patient" in output, output[-2000:]
