"""What an autotuning times (no GPU): the installed shape and the lattice's
default as whole shapes before anything else, and among the tiles every default
tile, so that a tuned context cannot come out slower than an untuned one."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_1701_07559_amd")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "ctx.h"
int main(int argc, char** argv) {
    using namespace mdwf;
    const mdwf_geometry geom{std::atoi(argv[1]), std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4]), 1};
    const mdwf_launch_tune none{{0, 0, 0, 0}, -1, -1, -1, -1, 0.0, -1};
    for (int p = 0; p < 3; ++p) {
        Geo g = plan_geo(geom, std::atoi(argv[5]));
        const mdwf_launch_tune own{{g.Xh, 2, 2, 1}, 0, 1, 2, 3, 0.0, 0};
        set_tune(g, Prec(p), own);
        for (const auto& t : tune_starts(g, Prec(p), none))
            std::printf("%d start %d,%d,%d,%d %d %d %d %d\n", p, t.tile[0], t.tile[1], t.tile[2], t.tile[3],
                        t.xcd_remap, t.nt_store, t.link_mode, t.rhs_group);
        for (const auto& b : tune_tiles(g)) std::printf("%d tile %d,%d,%d,%d\n", p, b[0], b[1], b[2], b[3]);
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc) or not os.path.exists(os.path.join(PKG, "libmdwf.so")):
        pytest.skip("needs hipcc and the built library")
    d = tmp_path_factory.mktemp("tune")
    src, exe = str(d / "tune.cpp"), str(d / "tune")
    with open(src, "w") as f:
        f.write(PROGRAM)
    r = subprocess.run([hipcc, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-Wno-unused-result", "-I", os.path.join(ROOT, "include"), "-I",
                        os.path.join(PKG, "csrc"), src, "-L" + PKG, "-lmdwf", "-Wl,-rpath," + PKG, "-o", exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.mark.parametrize("dims,L5,tile,group", [
    ((32, 32, 32, 64), 8, "16,16,8,2", "1 1 1"), ((20, 20, 20, 40), 10, "10,10,5,2", "1 1 1"),
    ((24, 24, 24, 64), 8, "12,12,6,2", "1 1 1"), ((16, 16, 16, 16), 8, "8,16,4,1", "1 1 1"),
    ((18, 18, 18, 24), 12, "9,18,2,1", "1 1 1"), ((30, 20, 24, 6), 5, "15,10,6,2", "2 2 2"), ((30, 20, 24, 6), 4, "15,10,6,2", "0 2 2")])
def test_the_default_is_timed(program, dims, L5, tile, group):
    out = subprocess.run([program] + [str(v) for v in dims + (L5,)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stderr
    lines = [l.split() for l in out.stdout.splitlines()]
    for p in range(3):
        starts = [l[2:] for l in lines if l[:2] == [str(p), "start"]]
        assert starts[0] == ["%d,2,2,1" % (dims[0] // 2), "0", "1", "2", "3"]
        assert starts[1:] == [[tile, "1", "1" if p == 2 else "0", "1", group.split()[p]]]
        assert tile in [l[2] for l in lines if l[:2] == [str(p), "tile"]]
