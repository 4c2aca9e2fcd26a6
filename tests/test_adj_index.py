"""The gravity adjoint's indices, which are built on the host (no GPU): a program over the library's own source checks
what the kernels rely on, for random task sets."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2008_05712_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists("/opt/rocm/include/hip/hip_runtime.h") or not shutil.which("g++"):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(tmp_path_factory.mktemp("adj") / "check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-x", "c++",
                           os.path.join(CSRC, "adj_index.hip"), os.path.join(ROOT, "tests", "adj_index_check.cpp"),
                           "-o", exe, "-pthread"])
    return exe


def test_items_and_records(program):
    out = subprocess.run([program], capture_output=True, text=True, timeout=100)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr


def test_a_build_without_memory(program):
    out = subprocess.run([program, "memory"], capture_output=True, text=True, timeout=100)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr
