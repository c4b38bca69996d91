"""Host-side rules of the library's persistent solves, called in the built
library from a small C++ program (no GPU): a launch never has more workgroups
than can be resident together."""
import os
import subprocess

import pytest

import paper_2106_01275_amd as dp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run(tmp_path, body):
    """Output of a program of the library's internals."""
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cmath>\n#include <cstdio>\n#include <cstring>\n#include "context.h"\nusing namespace dp;\n' + body)
    lib = os.path.dirname(dp.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(lib, "csrc"), "-I", "/opt/rocm/include", str(src), "-o", str(exe), dp.LIB_PATH,
                    f"-Wl,-rpath,{lib}", "-Wl,-rpath,/opt/rocm/lib", "-L/opt/rocm/lib", "-lamdhip64"], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout


@pytest.mark.parametrize("cus", [256, 128, 64, 32, 8, 1])
def test_groups_are_resident_together(tmp_path, cus):
    """Every lattice that the rule takes, on devices (or partitions of one) of
    several sizes: a group's workgroups cover its sites, all groups fit."""
    out = run(tmp_path, """
int main() {
    dp_ctx ctx;
    ctx.small_grid = %d;
    long taken = 0, bad = 0;
    for (int a = 1; a <= 34; a += a < 8 ? 1 : 3)
        for (int b = 1; b <= 34; b += a < 8 ? 1 : 3)
            for (int c = 1; c <= 16; ++c)
                for (int w = 1; w <= 256; w *= 2)
                    for (int eo = 0; eo < 2; ++eo) {
                        Lat L{{a, b, c, 4}, a * b * c * 4, eo};
                        SolveCfg cfg;
                        const int ns = eo ? L.N / 2 : L.N;
                        if (!small_problem(&ctx, L, 3, w, cfg)) continue;
                        ++taken;
                        const SmallShape z = small_shape(L, w, ctx.small_grid);
                        bad += z.nwg * 64 < ns || (z.nwg - 1) * 64 >= ns;
                        bad += z.nwg * z.ngroups > %d || z.ngroups < 1;
                        bad += z.wg != 1 && z.wg != 2 && z.wg != 4;
                    }
    std::printf("%%ld %%ld", taken, bad);
}""" % (cus, cus))
    taken, bad = (int(v) for v in out.split())
    assert taken > 20 and bad == 0
