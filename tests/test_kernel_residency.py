"""Waves per SIMD of the kernels whose dispatch lines count on them (from the compiler's report of the last build)."""
import os

import pytest

REPORT = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "_build", "kernel_resources.txt")

# mangled name up to the parameters: waves per SIMD
WAVES = {
    "_Z16br_k_route_splitILi4ELb0EE": 6, "_Z16br_k_route_splitILi4ELb1EE": 6,   # below 2048 clusters, two or three waves each
    "_Z16br_k_route_splitILi8ELb0EE": 5, "_Z16br_k_route_splitILi8ELb1EE": 5,
    "_Z10br_k_routeILi4ELi4EE": 6, "_Z10br_k_routeILi8ELi4EE": 5,               # 4097..6144 (5120) clusters with decode steps
    "_Z10br_k_routeILi4ELi8EE": 4, "_Z10br_k_routeILi8ELi8EE": 4,
    "_Z11br_k_assignILi4ELi0ELi4E": 6, "_Z11br_k_assignILi8ELi0ELi4E": 6,       # 5121..6144 clusters, no reductions
    "_Z11br_k_assignILi4ELi0ELi8E": 5, "_Z11br_k_assignILi8ELi0ELi8E": 5,
    "_Z11br_k_assignILi4ELi0ELi0ELb1ELb0E": 3, "_Z11br_k_assignILi8ELi0ELi0ELb1ELb0E": 3,   # BR-0, windows of 9..16
    "_Z11br_k_assignILi16ELi0ELi0ELb1ELb0E": 3,
}


@pytest.mark.skipif(not os.path.exists(REPORT), reason="no build report")
@pytest.mark.parametrize("name", sorted(WAVES))
def test_waves_per_simd(name):
    lines = [line for line in open(REPORT) if line.startswith(name)]
    assert len(lines) == 1, f"{name}: {len(lines)} kernels of that name in the report"
    got = int(lines[0].split("occupancy=")[1].split()[0])
    assert got >= WAVES[name], lines[0].strip()
