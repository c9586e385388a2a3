"""CPU test of the tile arithmetic that k_receiver_values and its launches share
(csrc/receiver_tiles.h): over the degrees, rank counts and forms of the receiver, every rank tile
and point tile is owned by exactly one wave, and every load a wave can issue lies inside the
buffer resource it goes through, scalar offset included (the hardware's range check does not cover
that offset, so a load past the end would read on into whatever follows)."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(__file__)), "paper_2605_15073_amd", "csrc")

PROGRAM = r"""
#include "receiver_tiles.h"
#include <cstdio>
#include <vector>
using namespace cgtp;

static long long bad = 0, loads = 0;
static void fail(const char *what, int lmax, int tiles, int half, int es, int a, int t)
{
    if (++bad <= 5) std::printf("%s: lmax %d tiles %d half %d es %d a %d t %d\n", what, lmax, tiles,
                                half, es, a, t);
}

int main()
{
    for (int lmax = 0; lmax <= 24; ++lmax)
        {
            const int U = (3 * lmax + 3) / 2, V = 3 * lmax + 1, UV = U * V;
            const int np = (UV + 31) / 32 * 2;  // point tiles of a row
            for (int tiles = 1; tiles <= 40; ++tiles)
                for (int half = 0; half < 2; ++half)
                    for (int es = 0; es < 2; ++es) {
                        RecvLaunch l[2];
                        const int n = recv_launches(tiles, half, es, l);
                        std::vector<int> owned((size_t)tiles * np, 0);
                        if (n < 1 || n > 2) fail("launches", lmax, tiles, half, es, n, 0);
                        for (int k = 0; k < n; ++k)
                            for (int g = 0; g < l[k].groups; ++g)
                                for (int p0 = 0; 16 * p0 < UV; p0 += l[k].pt) {
                                    const int rt0 = l[k].first + g * l[k].rt;
                                    const int na = wave_rank_tiles(l[k].rt, l[k].part, tiles, rt0);
                                    if (na < 1 || na > l[k].rt || rt0 + na > tiles)
                                        fail("rank tiles", lmax, tiles, half, es, na, p0);
                                    const unsigned bytes = value_bytes(na, np, p0);
                                    if ((long long)rt0 * np + p0 + bytes / 1024 > (long long)tiles * np)
                                        fail("resource", lmax, tiles, half, es, na, p0);
                                    for (int a = 0; a < na; ++a)
                                        for (int t = 0; t < l[k].pt; ++t) {
                                            ++loads;
                                            const int q = value_point_tile(l[k].pt, t, np, p0);
                                            if (q < 0 || value_offset(a, q, np) + 1024u > bytes)
                                                fail("load", lmax, tiles, half, es, a, t);
                                            if (p0 + t < np && rt0 + a < tiles) {
                                                if (q != t) fail("point", lmax, tiles, half, es, a, t);
                                                ++owned[(size_t)(rt0 + a) * np + p0 + t];
                                            }
                                        }
                                }
                        for (int r = 0; r < tiles; ++r)
                            for (int p = 0; 16 * p < UV; ++p)
                                if (owned[(size_t)r * np + p] != 1)
                                    fail("owners", lmax, tiles, half, es, r, p);
                    }
        }
    std::printf("%lld loads, %lld faults\n", loads, bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_receiver_tiles_stay_inside(tmp_path):
    src, exe = tmp_path / "tiles.cpp", tmp_path / "tiles"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout
