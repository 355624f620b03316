"""Positions of P^T's work ranges at the largest pixel a plan accepts (2^31 - 1 samples): the
header that the kernels use, compiled for the host."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WALK = r"""
#include <cinttypes>
#include <cstdio>
#include <initializer_list>
#include "mm_pos.h"
using namespace mm;
int main() {
    const int E = 4;
    for (int64_t n : {(int64_t)1, (int64_t)257, ((int64_t)1 << 30) + 5, ((int64_t)1 << 31) - 1}) {
        for (int64_t at : {(int64_t)0, (int64_t)63, ((int64_t)1 << 31) + 17}) {  // first sample
            const int64_t base = range_base(at, at + n);
            if (base & 63) return 9;
            const pos_t i0 = (pos_t)(at - base), i1 = (pos_t)(at + n - base);
            if (i0 + base != at || i1 + base != at + n) return 10;
            int64_t want = at & ~(int64_t)(E - 1), chunks = 0;
            for (pos_t c = first_chunk(i0, E); c < i1; c = next_chunk(c, E), want += 64 * E) {
                if (++chunks > n / (64 * E) + 2) return 1;                 // does not end
                if (c + base != want) return 2;
                if (next_chunk(next_chunk(c, E), E) + base != want + 128 * E) return 3;
                for (int lane : {0, 1, 63}) {
                    const pos_t b = lane_base(c, lane, E);
                    if (b + base != want + lane * E) return 4;
                    if ((b >> 6) + (base >> 6) != (want + lane * E) >> 6) return 5;
                    if ((b & 63) != ((want + lane * E) & 63)) return 6;
                    if (weight_index(b + E) + 2 * base != 2 * (want + lane * E + E)) return 7;
                }
            }
            if (want < at + n) return 8;
        }
    }
    return 0;
}
"""


@pytest.mark.skipif(os.system("g++ --version > /dev/null 2>&1") != 0, reason="no host compiler")
def test_positions_reach_the_largest_pixel(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fsanitize=undefined",
                    "-fno-sanitize-recover=undefined",
                    "-I", os.path.join(ROOT, "paper_1408_3048_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    assert subprocess.run([str(exe)], timeout=60).returncode == 0
