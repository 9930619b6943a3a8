"""Domains per work group, the unit lists and what decides between two,
three and four launches per iteration (paper_2411_06224_amd/csrc/planner.cpp:
group_domains, halo_units), so that the GPU tests on these systems do run the
branches they name.  The planner is compiled with a main of its own."""

import os
import subprocess

import numpy as np
import pytest

from group_systems import EDGES, SYSTEMS, line, system

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2411_06224_amd", "csrc")

MAIN = r"""
#include "planner.hpp"
#include <cstdio>
int main(int, char** argv) {
    FILE* f = fopen(argv[1], "rb");
    int h[3];
    if (!f || fread(h, 4, 3, f) != 3) return 1;
    std::vector<int> rp(h[0] + 1), ci(h[1]), gp(h[0] + 1), ga(h[2]);
    for (auto* v : {&rp, &ci, &gp, &ga})
        if (fread(v->data(), 4, v->size(), f) != v->size()) return 1;
    maspcg::Plan P;
    if (!maspcg::analyze(h[0], h[1], rp.data(), ci.data(), gp.data(), ga.data(), 16, 0, P).empty()) return 1;
    printf("%d %d %d %d %d %d\n", P.M, P.D0, P.halo ? 1 : 0, P.maxH, P.W1, P.GW);
}
"""


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    d = tmp_path_factory.mktemp("planner")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "probe")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                    str(d / "main.cpp"), os.path.join(CSRC, "planner.cpp"), "-o", exe, "-lpthread"], check=True)

    def run(s):
        p = str(d / "pattern")
        with open(p, "wb") as f:
            np.array([s.n, len(s.col_idx), len(s.gadj)], np.int32).tofile(f)
            for a in (s.row_ptr, s.col_idx, s.gptr, s.gadj):
                np.asarray(a, np.int32).tofile(f)
        out = subprocess.run([exe, p], check=True, capture_output=True, text=True).stdout
        return dict(zip(("M", "D0", "halo", "maxH", "W1", "GW"), map(int, out.split())))

    return run


@pytest.mark.parametrize("name", list(SYSTEMS))
def test_group_branches(probe, name):
    P = probe(system(name))
    assert P["M"] > 640  # more domains than groups the rule aims at: more than one per group where nothing is heavy
    assert P["D0"] == SYSTEMS[name][1]
    assert bool(P["halo"]) == SYSTEMS[name][2]
    # at most two passes of 256 threads over the group's writers: by recurrence
    assert P["W1"] <= 64 and 3 * P["GW"] <= 512


@pytest.mark.parametrize("n,domains", EDGES)
def test_group_size_edges(probe, n, domains):
    P = probe(line(n))
    assert P["M"] == n // 16
    assert P["D0"] == domains and P["halo"] == 1
