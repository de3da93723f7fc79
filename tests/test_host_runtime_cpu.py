"""The library's host side (plans, launch shapes, buffers, captured graphs) on
a HIP runtime of host memory and empty kernels: host_runtime.cpp, linked
against the built library, one scenario per test."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2103_01691_amd")
ROCM = os.path.dirname(os.path.dirname(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("host") / "host_runtime")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                        os.path.join(HERE, "host_runtime.cpp"), "-rdynamic", "-L", PKG, "-l:libmumode.so",
                        "-Wl,-rpath," + PKG, "-Wl,-rpath-link," + os.path.join(ROCM, "lib"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("scenario", ["batch_failed_rebuild", "resident_plans_fit", "flat_operators",
                                      "very_many_fibres", "oscillator_little_memory",
                                      "oscillator_failed_formation", "midpoint_little_memory",
                                      "tune_file_versions", "steps_per_launch"])
def test_host_runtime(program, scenario):
    r = subprocess.run([program, scenario], capture_output=True, text=True, timeout=300, cwd=os.path.dirname(program))
    assert r.returncode == 0, r.stdout + r.stderr
