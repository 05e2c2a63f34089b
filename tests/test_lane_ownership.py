"""Channels of k_scan_m's lanes (pgf_lane.h, plain arithmetic), on the CPU:
every channel's state and outputs are stored by exactly one wave, which
computes that channel, whatever the number of channels."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <stdio.h>
#include <vector>
#include "pgf_lane.h"
int main() {
    int bad = 0;
    for (int nc = 1; nc <= 4; nc *= 2)
        for (int D = 1; D <= 700; ++D) {
            std::vector<int> owner(D, -1);
            for (int w = 0; w * 16 * nc < D; ++w) {
                const int d0 = w * 16 * nc, skip = pgf::wave_skip(D, nc, d0);
                for (int c = 0; c < 16; ++c) {
                    const int first = pgf::lane_first(D, nc, d0, c);
                    if (first < 0 || (D >= nc && first + nc > D)) ++bad;
                    for (int j = 0; j < nc; ++j) {
                        if (!pgf::lane_stores(D, skip, j)) continue;
                        int &o = owner[first + j];
                        if (o >= 0 && o != w) { printf("nc %d D %d channel %d: waves %d and %d\n", nc, D, first + j, o, w); ++bad; }
                        o = w;
                    }
                }
            }
            for (int d = 0; d < D; ++d)
                if (owner[d] != d / (16 * nc)) { printf("nc %d D %d channel %d: wave %d\n", nc, D, d, owner[d]); ++bad; }
        }
    printf("%d faults\n", bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_each_channel_is_stored_by_one_wave(tmp_path):
    src, exe = tmp_path / "lane.cpp", tmp_path / "lane"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2512_23068_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("0 faults"), r.stdout[-2000:]
