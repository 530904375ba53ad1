"""The launch plans of dsq_conv2d_wq (CPU only: the planner's header in a small program): every
layer has one, their patches hold the rows of every tile, and planning takes no longer on wide rows."""
import os
import random
import subprocess

import pytest

from paper_1908_05033_amd import binding as B
from test_patch_plan import _rows_of_every_tile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(B.__file__)))

# One line "N C_in H W C_out R stride pad tile" in, one line "found TW PC npx lds microseconds" out.
PROGRAM = r"""
#include <chrono>
#include <cstdio>
#include "wq_plan.h"
int main()
{
    const WqTile tiles[] = {kSquare, kRow, kLarge, kNarrow, kSplit};
    DsqConvArgs a;
    int which;
    while (scanf("%d %d %d %d %d %d %d %d %d", &a.N, &a.C_in, &a.H, &a.W, &a.C_out, &a.R, &a.stride, &a.pad, &which) == 9) {
        a.Ho = (a.H + 2 * a.pad - a.R) / a.stride + 1;
        a.Wo = (a.W + 2 * a.pad - a.R) / a.stride + 1;
        WqPlan pl = {};
        int lds = 0;
        bool found = false;
        double best = 1e9;
        for (int i = 0; i < 5; ++i) {
            const auto t = std::chrono::steady_clock::now();
            for (int k = 0; k < 20; ++k) found = plan_wq(a, tiles[which], pl, lds);
            const double us = std::chrono::duration<double>(std::chrono::steady_clock::now() - t).count() * 1e6 / 20;
            best = us < best ? us : best;
        }
        printf("%d %d %d %d %d %f\n", (int)found, pl.TW, pl.PC, pl.npx, lds, best);
    }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("wq_plan")
    (d / "plan.cpp").write_text(PROGRAM)
    lib = os.path.dirname(B.LIB_PATH)
    cmd = ["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(lib, "csrc"),
           str(d / "plan.cpp"), "-o", str(d / "plan"), "-L" + lib, "-l:libdsqconv.so", "-L/opt/rocm/lib", "-lamdhip64",
           "-Wl,-rpath," + lib, "-Wl,-rpath,/opt/rocm/lib"]
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert proc.returncode == 0, proc.stdout[-2000:]

    def run(cases):
        text = "\n".join(" ".join(map(str, c)) for c in cases) + "\n"
        out = subprocess.run([str(d / "plan")], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout.split("\n")
        rows = [r.split() for r in out if r]
        assert len(rows) == len(cases)
        return [tuple(map(int, r[:5])) + (float(r[5]),) for r in rows]
    return run


BP = (64, 64, 128, 128, 32)
SPLIT = 4


def test_every_layer_has_a_plan_that_holds_its_tiles(plan):
    rng = random.Random(5)
    cases = []
    while len(cases) < 400:
        R, stride = rng.choice([1, 3, 3, 3]), rng.choice([1, 2])
        pad = rng.randint(0, R - 1)
        H, W = rng.choice([1, 2, 3, rng.randint(1, 90)]), rng.choice([1, 2, 3, rng.randint(1, 90), rng.randint(1, 700)])
        if min(H, W) + 2 * pad >= R:
            cases.append((rng.choice([1, 2, 7, 64]), 20, H, W, 40, R, stride, pad, rng.randrange(5)))
    for c, (found, TW, PC, npx, lds, _) in zip(cases, plan(cases)):
        N, _, H, W, _, R, stride, pad, tile = c
        assert found or tile != SPLIT, c
        if not found:
            continue
        assert lds <= 160 * 1024
        if R == 3:
            Ho = (H + 2 * pad - R) // stride + 1
            assert npx >= PC * _rows_of_every_tile(N, H, Ho, stride, pad, R, TW, BP[tile]), c
            assert PC == (TW - 1) * stride + R


@pytest.mark.parametrize("H,W", [(3, 4096), (3, 30000), (16, 2048), (64, 1024)])
def test_planning_time_of_wide_rows(plan, H, W):
    """Rows far wider than any patch cost no more to plan than a few ordinary layers (20 to 100 times
    the 3x224 layer's time when every width was counted)."""
    ordinary = max(r[5] for r in plan([(1, 64, 3, 224, 64, 3, 1, 1, t) for t in range(5)]))
    wide = max(r[5] for r in plan([(1, 64, H, W, 64, 3, 1, 1, t) for t in range(5)]))
    assert wide < 10 * ordinary, (wide, ordinary)
