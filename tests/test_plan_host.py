"""The plan's host code over a HIP runtime that lives on the host (tests/plan_host.cpp): which
device its lists are put on, what a shortage of host memory does, and shapes chosen by several
threads."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1905_00934_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if shutil.which("g++") is None or not os.path.isdir(os.path.join(rocm, "include", "hip")):
        pytest.skip("g++ or the HIP headers are not available")
    exe = str(tmp_path_factory.mktemp("ph") / "plan_host")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-pthread", "-D__HIP_PLATFORM_AMD__",
           "-I", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(ROOT, "tests", "plan_host.cpp"), os.path.join(CSRC, "plan.cpp"),
           "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def _run(program, what):
    r = subprocess.run([program, what], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout + r.stderr


def test_projector_lists_are_on_the_plans_device(program):
    _run(program, "device")


def test_projector_lists_without_host_memory(program):
    _run(program, "nomem")


def test_launch_shapes_chosen_by_several_threads(program):
    _run(program, "threads")
