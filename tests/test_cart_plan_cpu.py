"""The marching step's plan against the waves that its LDS allows (host code only,
compiled here from the planner's header)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FP64, FP32DEV, FP32NEQ = 0, 1, 2

PROGRAM = r"""
#define __HIP_PLATFORM_AMD__
#include "cart_plan.h"
#include <cstdio>
using namespace sdg;
int main()
{
    int nx, ny, per, n_bc, mode;
    while (std::scanf("%d %d %d %d %d", &nx, &ny, &per, &n_bc, &mode) == 5) {
        DevCart c{};
        c.nx = nx; c.ny = ny; c.per_x = per & 1; c.per_y = per >> 1;
        const CartPlan p = plan_march({c}, n_bc, mode);
        const CartTimes t = cart_times(mode);
        cart_cut(c, p.rows);
        std::printf("%d %d %d %.9g %.9g %.9g\n", c.strips, c.segs, c.seg_h + (c.seg_more > 0), p.us, t.launch, t.row[0]);
    }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(PROGRAM)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2007_07347_amd", "csrc"),
                    "-I", os.path.join(rocm, "include"), str(src), "-o", str(exe)], check=True)

    def call(rows):
        text = "\n".join(" ".join(map(str, r)) for r in rows)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
        return [[float(x) for x in line.split()] for line in out.splitlines()]
    return call


def test_planned_rounds_are_those_the_lds_allows(plan):
    """A CU holds as many waves as its 160 KB of LDS (in units of 1280 bytes) do,
    eight at most.  A plan's time is at least that of its rounds, each at least a row's
    time with one wave on a SIMD for every row of the longest segment."""
    rows = [(n, m, per, n_bc, mode) for n in (64, 700, 1600, 1792, 2048, 2560, 4096) for m in (40, 1024, 2048, 5000)
            for per in (0, 1, 2, 3) for n_bc in (0, 2, 64) for mode in (FP64, FP32DEV, FP32NEQ) if n_bc or per == 3]
    for (nx, ny, per, n_bc, mode), (strips, segs, seg_h, us, launch, row) in zip(rows, plan(rows)):
        ring = 3 * 64 * (3 * 8 + 9 * (8 if mode == FP64 else 4))
        value = 4 if mode == FP32DEV else 8
        columns = 0 if per & 1 else (2 if strips == 1 else 1)
        lds = ring + 32 * n_bc + columns * (seg_h + 4) * 9 * value
        at_once = 256 * min(8, 160 * 1024 // (-(-lds // 1280) * 1280))
        rounds = -(-strips * segs // at_once)
        assert us >= launch + rounds * row * seg_h, (nx, ny, per, n_bc, mode, strips, segs, seg_h, lds, at_once, us)
