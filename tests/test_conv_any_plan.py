"""The launch shapes of the ragged convolution, over every channel count it
takes and grids of all sizes, on the CPU: the block's LDS, the weight pieces
that its threads hold between stages, and the cover of grid and channels."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cstdio>
#include "conv_any_plan.hpp"
int main() {
    const int n[] = {1, 2, 3, 4, 5, 8, 10, 14, 17, 24, 31, 40, 44, 56, 64, 72, 88, 104, 120, 200};
    long plans = 0, staged = 0, bad = 0;
    for (int cin = 16; cin <= 144; cin += 16)
        for (int cout = 16; cout <= 192; cout += 16)
            for (int nx : n) for (int ny : n) for (int nz : n) for (long cus : {64L, 256L}) {
                const AnyPlan p = any_plan(cin, cout, nx, ny, nz, cus);
                ++plans;
                if (cin > 128) {
                    bad += p.mt != 0;
                    continue;
                }
                const long tx = 1L << p.ltx, ty = 16 * p.mt >> p.ltx;
                const size_t row = 2 * cin + 16, hp = (tx + 2) * (ty + 2) * 6;
                const bool in_lds = p.lds == hp * row + (size_t)p.taps * 16 * p.nt * row && p.lds <= 160 * 1024;
                const bool taps = p.taps == 3 || p.taps == 9 || p.taps == 27;
                const bool held = p.taps == 27 || p.taps * 16 * p.nt * (cin / 8) <= 256 * any_pieces(cin / 16, p.nt);
                const bool cover = p.ntile == ((nx + tx - 1) / tx) * ((ny + ty - 1) / ty) * ((nz + 3) / 4) &&
                                   cout % (16 * p.nt) == 0 && tx * ty == 16 * p.mt;
                staged += p.taps < 27;
                if (!(p.mt > 0 && in_lds && taps && held && cover)) {
                    if (!bad++) std::printf("%d -> %d on %d x %d x %d\n", cin, cout, nx, ny, nz);
                }
            }
    std::printf("%ld plans, %ld staged, %ld bad\n", plans, staged, bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_plans_fit_the_kernel(tmp_path):
    (tmp_path / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2407_12263_amd", "csrc"), "-o", str(tmp_path / "plans"),
                    str(tmp_path / "main.cpp")], check=True)
    r = subprocess.run([str(tmp_path / "plans")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
