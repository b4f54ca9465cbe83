"""How k_grouped_stream deals the tiles of crowded experts to its workgroups.

A program of its own is compiled for the host from the header that the kernel takes it from.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "moe_deal.h"
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

struct Result { int wrong, most, least; };

// every tile to one workgroup and one alone; the most and the fewest tiles that a workgroup which takes both kinds has
Result check(int n_whole, int n_rest, int nt, int K)
{
    std::vector<int> whole(size_t(n_whole) * nt), rest(size_t(n_rest) * nt);
    Result r = {0, 0, 1 << 30};
    for (int w = 0; w < StreamDeal::WORKGROUPS; ++w) {
        const StreamDeal d(w, n_whole, n_rest, nt, K);
        auto note = [&](std::vector<int>& seen, int n, StreamDeal::Place at) {
            if (at.row < 0 || at.row >= n || at.column < 0 || at.column >= nt) ++r.wrong;
            else ++seen[size_t(at.row) * nt + at.column];
        };
        for (int s = 0; s < d.whole_count(); ++s) note(whole, n_whole, d.whole(s));
        for (int s = 0; s < d.rest_count(); ++s) note(rest, n_rest, d.rest(s));
        const int all = d.whole_count() + d.rest_count();
        if (d.leave && (w >> 3) >= 28) { r.wrong += d.rest_count() != 0; continue; }
        r.most = std::max(r.most, all);
        r.least = std::min(r.least, all);
    }
    for (int n : whole) r.wrong += n != 1;
    for (int n : rest) r.wrong += n != 1;
    return r;
}

int main()
{
    int wrong = 0, uneven = 0, leaves = 0;
    unsigned state = 1;
    auto draw = [&](int n) { state = state * 1664525u + 1013904223u; return int((state >> 8) % unsigned(n)); };
    for (int i = 0; i < 6000; ++i) {
        const int n_whole = draw(3) ? draw(i % 3 ? 12 : 300) : draw(2), n_rest = draw(3) ? draw(i % 4 ? 40 : 1500) : draw(2), nt = 1 + draw(i % 5 ? 9 : 33), K = 64 * (4 + draw(60));
        const Result r = check(n_whole, n_rest, nt, K);
        wrong += r.wrong;
        uneven = std::max(uneven, r.most - r.least);
        leaves += StreamDeal(0, n_whole, n_rest, nt, K).leave;
    }
    const Result largest = check(0, 4096, 32, 256);            // as many tiles of a kind as a workgroup can have
    std::printf("%d %d %d %d\n", wrong + largest.wrong, uneven, leaves, largest.most);
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_every_tile_goes_to_one_workgroup(tmp_path):
    source, program = tmp_path / "deal.hip", tmp_path / "deal"
    source.write_text(SOURCE)
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-function",
                    "-I", os.path.join(ROOT, "paper_1707_02402_amd", "csrc"), "-x", "hip", str(source), "-o", str(program)], check=True, capture_output=True, timeout=300)
    wrong, uneven, leaves, largest = map(int, subprocess.run([str(program)], check=True, capture_output=True, text=True, timeout=60).stdout.split())
    assert wrong == 0
    assert uneven <= 3                                         # shares of a list that differ by a tile a team, in both lists, and the round that is cut short
    assert leaves > 200                                        # both sides of the rule
    assert largest == 586
