"""The arithmetic with which the general convolution kernels find a step's tap, in every panel that a launch can choose.

Panels of many steps belong to maps of a few pixels with thousands of channels, whose weights take gigabytes; the arithmetic needs
none of them.  A program of its own is compiled for the host from the kernels' header.
"""
import os
import shutil
import subprocess

import pytest

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
    // a join with both arguments in LDS: as many steps as fit beside one pixel; a 3x3 stages at least the nine of a 1 x 1 map
    int largest2 = 0, largest9 = 0, wrong = 0;
    for (int nj = 1; 2ll * conv_pixel_bytes(nj * 16, 4) <= CONV_LDS_BOTH; ++nj) { wrong += walk<2>(nj); largest2 = nj; }
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
    assert largest2 == 1279 and 120 <= largest9 <= 142      # the panels that the launches' limits on LDS allow
    assert wrong == 0
