"""The hash under which bench.py takes committed counters covers every source that the traced
kernels and their launch orders are built from."""
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_1905_00934_amd", "csrc")


def _closure(name, seen):
    if name in seen or not os.path.exists(os.path.join(CSRC, name)):
        return
    seen.add(name)
    with open(os.path.join(CSRC, name), encoding="utf-8") as f:
        for inc in re.findall(r'^#include "([^"]+)"', f.read(), re.M):
            _closure(inc, seen)


def test_counters_hash_covers_the_kernels():
    need = set()
    for unit in ("tomo.hip", "udm.hip", "admm.hip", "fft.hip", "plan.cpp"):
        _closure(unit, need)
    need.discard("profile.h")  # event timing around the launches
    assert need <= set(bench.KERNEL_SOURCES)
