"""The projector's workgroup lists checked on the host (tests/projector_balance.cpp, built with
g++ from the plan's own projorder.h): no XCD has much more than its share of a launch."""
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
    "ragged_fan": S.geometry("fan", 37, 29, 0.4, 50, 71, 0.45, det_offset=0.3, src_iso_cm=30.0,
                             src_det_cm=52.0, angle0=0.1),
    "sym_fan_offset": S.geometry("fan", 32, 32, 0.5, 44, 57, 0.6, det_offset=0.37,
                                 src_iso_cm=30.0, src_det_cm=50.0, angle0=0.2),
    "one_view": S.geometry("parallel", 7, 5, 0.5, 1, 9, 0.5, angle0=0.3),
    "one_bin": S.geometry("fan", 6, 6, 0.5, 12, 1, 0.4, src_iso_cm=12.0, src_det_cm=20.0),
    "odd_fan101": S.fan_geometry_fov(101, 121, 161),
    "fan160": S.fan_geometry_fov(160, 224, 320),
    "fan256": S.fan_geometry_fov(256, 360, 512),
}


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("pl") / "projector_balance")
    cmd = ["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_1905_00934_amd", "csrc"),
           os.path.join(ROOT, "tests", "projector_balance.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("name", list(CASES))
def test_no_xcd_has_more_than_its_share(checker, name):
    g = CASES[name]
    full = abs(g["span"] - 2 * math.pi) < 1e-12
    sym = 4 if (g["kind"] == "fan" and full and g["n_views"] % 4 == 0 and g["nx"] == g["ny"]
                and g["nx"] % 2 == 0) else 1
    args = [str(v) for v in (0 if g["kind"] == "parallel" else 1, g["nx"], g["ny"],
                             g["pixel_cm"], g["n_views"], g["n_det"], g["det_cm"],
                             g["det_offset"], g["src_iso_cm"], g["src_det_cm"], g["angle0"],
                             g["span"], sym)]
    r = subprocess.run([checker, *args], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.strip().endswith("OK")
