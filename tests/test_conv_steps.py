"""The arithmetic with which the general convolution kernels find a step's tap, in every panel that a launch can choose.

Panels of many steps belong to maps of a few pixels with thousands of channels, whose weights take gigabytes; the arithmetic needs
none of them.  A program of its own is compiled for the host from the kernels' header.  The registers that the kernels take are
read from the library's own build.
"""
import os
import shutil
import subprocess

import pytest

from tests.test_handover import OBJDUMP, code_objects

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PACKAGE = os.path.join(ROOT, "paper_1707_02402_amd")

SOURCE = r"""
#include "iep_conv.h"
#include <cstdio>

template <int TAPS> int walk(int nj)
{
    int wrong = 0;
    for (int s = 0; s < TAPS * nj; ++s)
        if (tap_of<TAPS>(s, nj, recip20_of(uint32_t(nj))) != s / nj) ++wrong;
    return wrong;
}

int main()
{
    // a join with both arguments in LDS: as many steps as fit it beside one pixel; a 3x3 stages at least the nine of a 1 x 1 map
    int largest2 = 0, largest9 = 0, wrong = 0;
    for (int nj = 1; 2ll * conv_pixel_bytes(nj * 16, 4) <= 160 * 1024; ++nj) { wrong += walk<2>(nj); largest2 = nj; }
    for (int steps = 1; steps <= 4096; ++steps) {
        ConvArgs a = {};
        a.C = steps * 16;
        a.H = a.W = a.sw = 1;
        const int nj = conv_panel<1, 4>(a) / 16;
        if (nj > largest9) { wrong += walk<9>(nj); largest9 = nj; }
    }
    // ... and k_node both of its tiles, whole
    for (int nj = 1; 2ll * 9 * conv_pixel_bytes(nj * 16, 4) <= 160 * 1024; ++nj) { wrong += walk<9>(nj); largest9 = nj > largest9 ? nj : largest9; }
    std::printf("%d %d %d\n", largest2, largest9, wrong);
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_tap_of_every_step_of_every_panel(tmp_path):
    source, program = tmp_path / "steps.hip", tmp_path / "steps"
    source.write_text(SOURCE)
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-function",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PACKAGE, "csrc"), "-x", "hip", str(source), "-o", str(program)],
                   check=True, capture_output=True, timeout=300)
    largest2, largest9, wrong = map(int, subprocess.run([str(program)], check=True, capture_output=True, text=True, timeout=60).stdout.split())
    assert largest2 == 1279 and 120 <= largest9 <= 142      # the panels that a CU's LDS allows
    assert wrong == 0


@pytest.mark.parametrize("mode,tile", [(0, "42"), (1, "42"), (1, "22"), (2, "22"), (4, "22"), (5, "42"), (5, "22"), (6, "42"), (6, "22")])
def test_three_workgroups_of_a_fp32_tile_fit_the_registers_of_a_cu(tmp_path, mode, tile):
    """At most 168 registers and none spilled, in every variant of the kernel that whole steps run (512 registers a SIMD, three waves)."""
    name = "k_convIfLNS_8ConvModeE%dELi%sELi%sELb1E" % (mode, *tile)
    seen = 0
    for path in code_objects(tmp_path):
        table = subprocess.run([OBJDUMP, "-t", path], check=True, capture_output=True, text=True).stdout
        value = {line.split()[-1]: int(line.split()[0], 16) for line in table.splitlines() if name in line}
        for symbol in value:
            if symbol.endswith(".num_vgpr"):
                assert value[symbol] + value[symbol.replace(".num_vgpr", ".num_agpr")] <= 168, symbol
                assert value[symbol.replace(".num_vgpr", ".private_seg_size")] == 0, symbol
                seen += 1
    assert seen >= 1
