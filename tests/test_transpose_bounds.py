"""The transposed projector's staged windows checked on the host with the kernel's own
arithmetic (tests/transpose_bounds.cpp, built with g++ from bpidx.h): every bin with a
nonzero weight on a pixel is among the candidates that the pixel takes, and every candidate
lies inside the staged window.  Parallel and fan beams, even, odd and ragged sizes, shifted
and narrow detectors, magnifications from bins wider than a pixel to many bins per pixel."""
import math
import os
import shutil
import subprocess

import pytest

from paper_1905_00934_amd import synth as S

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CASES = {
    "tiny_parallel": S.geometry("parallel", 64, 64, 0.5, 90, 95, 0.5),
    "ragged_parallel": S.geometry("parallel", 33, 47, 0.5, 41, 300, 0.17, det_offset=-0.25,
                                  angle0=0.05),
    "wide_bins": S.geometry("parallel", 40, 40, 0.5, 23, 21, 1.6),
    "narrow_detector": S.geometry("parallel", 50, 46, 0.5, 31, 17, 0.5, det_offset=3.0),
    "ragged_fan": S.geometry("fan", 37, 29, 0.4, 50, 71, 0.45, det_offset=0.3, src_iso_cm=30.0,
                             src_det_cm=52.0, angle0=0.1),
    "near_source": S.geometry("fan", 48, 48, 0.5, 60, 200, 0.5, src_iso_cm=20.0, src_det_cm=45.0),
    "sym_fan_offset": S.geometry("fan", 32, 32, 0.5, 44, 57, 0.6, det_offset=0.37,
                                 src_iso_cm=30.0, src_det_cm=50.0, angle0=0.2),
    "sym_near_source": S.geometry("fan", 36, 36, 0.5, 48, 150, 0.5, src_iso_cm=15.0,
                                  src_det_cm=30.0),
    "two_by_two": S.geometry("parallel", 2, 2, 1.0, 7, 5, 0.8),
    "two_by_two_fan": S.geometry("fan", 2, 2, 1.0, 8, 5, 0.8, src_iso_cm=10.0, src_det_cm=18.0),
    "two_by_two_fan_close": S.geometry("fan", 2, 2, 1.0, 8, 9, 0.4, src_iso_cm=3.5,
                                       src_det_cm=8.0),
    "fan256": S.fan_geometry_fov(256, 360, 512),
    "fan512": S.fan_geometry_fov(512, 720, 1024),
}


def _sym(g):
    full = abs(g["span"] - 2 * math.pi) < 1e-12
    return 4 if (g["kind"] == "fan" and full and g["n_views"] % 4 == 0 and g["nx"] == g["ny"]
                 and g["nx"] % 2 == 0) else 1


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("tb") / "transpose_bounds")
    cmd = ["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_1905_00934_amd", "csrc"),
           os.path.join(ROOT, "tests", "transpose_bounds.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("name", list(CASES))
def test_candidates_cover_every_weight(checker, name, prec):
    g = CASES[name]
    kind = 0 if g["kind"] == "parallel" else 1
    args = [str(v) for v in (kind, g["nx"], g["ny"], g["pixel_cm"], g["n_views"], g["n_det"],
                             g["det_cm"], g["det_offset"], g["src_iso_cm"], g["src_det_cm"],
                             g["angle0"], g["span"], _sym(g), prec)]
    r = subprocess.run([checker, *args], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip().endswith("OK")
