"""Waves per SIMD of the BR-H kernels, and no scratch memory in them (from the compiler's report of the last build): a batch of 4096
clusters of one wave each is four waves per SIMD."""
import os

import pytest

REPORT = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "_build", "kernel_resources.txt")

# mangled name up to the parameters: waves per SIMD.  <4, ...>: queues of up to 256, <8, ...>: 512; <., 4>: H <= 4, <., 8>: H <= 8
WAVES = {
    "_Z11br_k_assignILi4ELi4ELi0ELb0ELb0E": 5, "_Z11br_k_assignILi8ELi4ELi0ELb0ELb0E": 4,   # no reductions
    "_Z11br_k_assignILi4ELi8ELi0ELb0ELb0E": 4, "_Z11br_k_assignILi8ELi8ELi0ELb0ELb0E": 4,
    "_Z12br_k_route_hILi4ELi4ELb0E": 5, "_Z12br_k_route_hILi8ELi4ELb0E": 4,                 # with reductions
    "_Z12br_k_route_hILi4ELi8ELb0E": 4, "_Z12br_k_route_hILi8ELi8ELb0E": 4,
    "_Z12br_k_route_hILi4ELi4ELb1E": 4, "_Z12br_k_route_hILi8ELi4ELb1E": 4,                 # and decode steps
    "_Z12br_k_route_hILi4ELi8ELb1E": 4, "_Z12br_k_route_hILi8ELi8ELb1E": 4,
    "_Z17br_k_route_helpedILi4ELi4E": 5, "_Z17br_k_route_helpedILi8ELi4E": 5,               # below 2048 clusters
    "_Z17br_k_route_helpedILi4ELi8E": 4, "_Z17br_k_route_helpedILi8ELi8E": 4,
    "_Z16br_k_assign_longILi4ELi4ELi0E": 4, "_Z16br_k_assign_longILi4ELi2ELi0E": 4, "_Z16br_k_assign_longILi4ELi1ELi0E": 4,
    "_Z20br_k_project_advanceILi32ELi4ELb1ELi0E": 8, "_Z20br_k_project_advanceILi16ELi8ELb1ELi0E": 5,
    "_Z20br_k_project_advanceILi32ELi8ELb1ELi0E": 5, "_Z20br_k_project_advanceILi64ELi8ELb1ELi0E": 4,
}


@pytest.mark.skipif(not os.path.exists(REPORT), reason="no build report")
@pytest.mark.parametrize("name", sorted(WAVES))
def test_waves_per_simd(name):
    lines = [line for line in open(REPORT) if line.startswith(name)]
    assert lines, f"no kernel {name} in the report"
    for line in lines:
        assert int(line.split("occupancy=")[1].split()[0]) >= WAVES[name] and line.rstrip().endswith("scratch=0"), line.strip()
