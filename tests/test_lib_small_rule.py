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
    src.write_text('#include <array>\n#include <cmath>\n#include <cstdio>\n#include <cstring>\n#include "context.h"\nusing namespace dp;\n' + body)
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


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_steps_to_the_next_check_are_bounded(tmp_path, prec):
    """A lane that hardly decays asks for the most steps, not for one: whatever
    the pace (down to the smallest number) the answer lies in 1 .. 32, and never
    grows with it."""
    out = run(tmp_path, """
int main() {
    const int prec = %d;
    long bad = 0;
    for (double ratio : {1e24, 1e12, 1e3, 1.5, 1.0, 0.0}) {
        int last = 32;
        for (double pace = 5e-324; pace < 100; pace = pace < 1e-300 ? pace * 1e8 + 1e-308 : pace * 1.7) {
            for (int mult : {1, 2})
                for (double mean : {0.1, 4.0}) {
                    Pace pc;
                    pc.last = pace;
                    pc.mean = mean;
                    const int n = plan_steps(pc, ratio, std::max(ratio, 1.0), 0.0, prec, mult);
                    const int most = mean > 1.7 || prec == kBF16 ? 32 : 16 / mult;
                    bad += n < 1 || n > most;
                    bad += ratio >= 1e3 && pace < 1e-6 && n != most;
                    if (mult == 1 && mean > 1.7) {
                        bad += n > last;
                        last = n;
                    }
                }
        }
    }
    // (the multi-instance engine's: 2 .. 16)
    for (double near = 1e-16; near < 0.5; near *= 3) bad += next_check(8, 1e20 * (1 - near), 1e20, 4, 0.0) != 16;
    bad += next_check(8, 10.0, 1e9, 4, 0.0) != 2;
    std::printf("%%ld", bad);
}""" % prec)
    assert int(out) == 0
