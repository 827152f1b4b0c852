"""Host C++ unit tests (tests/host_cpp/test_step.cpp) of the step kernels'
host-side rules, built with g++ against the library and run on the CPU."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm"


def run_units(tmp_path, *args):
    gxx = shutil.which("g++")
    lib = os.path.join(ROOT, "paper_2502_12350_amd", "libwfd.so")
    if gxx is None or not os.path.isdir(os.path.join(ROCM, "include")):
        pytest.skip("g++ or the HIP headers not available")
    exe = str(tmp_path / "test_step")
    cmd = [gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__",
           "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2502_12350_amd", "csrc"),
           os.path.join(ROOT, "tests", "host_cpp", "test_step.cpp"), lib,
           "-L", os.path.join(ROCM, "lib"), "-lamdhip64",
           f"-Wl,-rpath,{os.path.dirname(lib)}", f"-Wl,-rpath,{ROCM}/lib", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "ALL PASSED" in r.stdout


def test_step_host_units(tmp_path):
    run_units(tmp_path)
