"""Which kernels a frame's plan takes (CPU only): a small host program reads
the plans of the library as it is built and prints their routes."""
import os
import subprocess

import pytest

from conftest import ROOT
from paper_1610_04121_amd import build, sgm

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include "sgm_plan.h"
// argv: groups of W H D P1 P2 paths flags(1 csct, 2 adaptive, 4 fused, 8 final pass)
int main(int argc, char** argv) {
    for (int i = 1; i + 6 < argc; i += 7) {
        auto v = [&](int k) { return std::atoi(argv[i + k]); };
        sgm::Plan p;
        p.W = v(0), p.H = v(1), p.D = v(2), p.P1 = v(3), p.P2 = v(4), p.n_paths = v(5);
        p.csct = v(6) & 1, p.adaptive = v(6) & 2, p.lrcheck = p.median = true;
        const char* why = "";
        if (!sgm::plan_finish(p, &why)) return 1;
        p.fused = v(6) & 4, p.final_pass = v(6) & 8;
        int gh = 0, gv = 0;
        sgm::default_lanes(p, &gh, &gv);
        std::printf("%d %d %d %d %d %d %zu\n", p.l16, sgm::fused_aggregation(p), sgm::final_pass_active(p),
                    sgm::row_kernel_active(p, false), gh, gv, sgm::workspace_bytes(p));
    }
}
"""
CSCT, ADAPTIVE, FUSED, FINAL = 1, 2, 4, 8


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    if not os.path.exists(sgm.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    d = tmp_path_factory.mktemp("routes")
    src, exe = d / "routes.cpp", d / "routes"
    src.write_text(SOURCE)
    subprocess.run([build.HIPCC, "-std=c++17", "--offload-arch=gfx950", "-I", os.path.join(ROOT, "paper_1610_04121_amd", "csrc"),
                    str(src), "-L" + os.path.dirname(sgm.LIB_PATH), "-l:" + os.path.basename(sgm.LIB_PATH),
                    "-Wl,-rpath," + os.path.dirname(sgm.LIB_PATH), "-o", str(exe)], check=True, capture_output=True)

    def run(*plans):
        out = subprocess.run([str(exe), *[str(x) for p in plans for x in p]], check=True, capture_output=True, text=True).stdout
        keys = ("l16", "fused", "final", "row", "gh", "gv", "bytes")
        return [dict(zip(keys, map(int, line.split()))) for line in out.splitlines() if line[0].isdigit()]
    return run


def test_final_pass_runs_where_a_byte_holds_the_summed_path_cost(routes):
    # (Cmax 62, CSCT 31): past it the plain route is the faster one
    for cmax, flag in ((62, 0), (31, CSCT)):
        at, past, p2_255, p2_256 = routes(*[(640, 480, 128, 7, P2, 4, FINAL | flag) for P2 in (255 - cmax, 256 - cmax, 255, 256)])
        assert at["final"] == 1
        assert past["final"] == p2_255["final"] == p2_256["final"] == 0
        assert [r["l16"] for r in (at, past, p2_255, p2_256)] == [0, 0, 0, 1]


def test_census_computing_aggregation_takes_the_fewest_levels_per_lane(routes):
    for W, H, P2, P in ((640, 480, 86, 4), (1000, 600, 86, 4), (1000, 600, 300, 8), (320, 240, 300, 2)):
        (r,) = routes((W, H, 256, 7, P2, P, FUSED))
        assert (r["fused"], r["gh"], r["gv"]) == (1, 64, 32)


def test_workspace_does_not_depend_on_the_plane_type_chosen(routes):
    # past Cmax + P2 = 255 the planes had 16 bits each
    a, b, c = routes(*[(640, 480, 128, 7, P2, 4, 0) for P2 in (193, 194, 256)])
    assert b["bytes"] == c["bytes"] > a["bytes"]
    assert (a["l16"], b["l16"], c["l16"]) == (0, 0, 1)
