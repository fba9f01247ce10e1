"""The staged projector checked on the host, one and two rays per lane, for every workgroup,
wave, lane and ray of a launch (tests/projector_lines.cpp, built with g++ from the kernel's own
helpers and the plan's own workgroup lists): windows, zero-extended line loads, taps, coverage."""
import os
import shutil
import subprocess

import pytest

from paper_1905_00934_amd import synth as S
from test_projector_bounds import CASES as GPU_CASES, ROOT, _sym

CASES = dict(GPU_CASES)
CASES.update({
    # Rays exactly on and one line beside the columns; four pixels to a bin; tiles of both axes.
    "on_columns_f64": (S.geometry("parallel", 9, 6, 0.5, 1, 11, 0.5), 64),
    "coarse_parallel_f32": (S.geometry("parallel", 24, 24, 0.1, 40, 33, 0.4), 32),
    "high_parallel_f32": (S.geometry("parallel", 35, 70, 0.5, 33, 230, 0.19, angle0=0.1), 32),
    "odd_fan101_f32": (S.fan_geometry_fov(101, 61, 161), 32),
})


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("pn") / "projector_lines")
    cmd = ["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_1905_00934_amd", "csrc"),
           os.path.join(ROOT, "tests", "projector_lines.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("name", list(CASES))
def test_staged_lines_and_taps(checker, name):
    g, prec = CASES[name]
    kind = 0 if g["kind"] == "parallel" else 1
    args = [str(v) for v in (kind, g["nx"], g["ny"], g["pixel_cm"], g["n_views"], g["n_det"],
                             g["det_cm"], g["det_offset"], g["src_iso_cm"], g["src_det_cm"],
                             g["angle0"], g["span"], _sym(g), prec)]
    r = subprocess.run([checker, *args], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip().endswith("OK")
