"""The default tiling (csrc/tuning.h, host code) over sizes and limits: the
choice keeps to the tiles that a caller has room for wherever the tiling by
the grid's size alone would, and is the unlimited choice where that fits."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = r"""
#include "tuning.h"
#include <cstdio>
#include <utility>
using namespace ofm;

static int64_t tiles(const TileChoice& t, int nd, const int* n, int count)
{
    int64_t k = 0;
    for (int i = 0; i < count; ++i)
        k += (int64_t)((n[i] + t.tx - 1) / t.tx) * (nd < 2 ? 1 : (n[i] + t.ty - 1) / t.ty) *
             (nd < 3 ? 1 : (n[i] + t.zchunk - 1) / t.zchunk);
    return k;
}

int main()
{
    const Tuning tuning;
    long bad = 0, held = 0, all = 0;
    auto check = [&](int prec, int nd, const int* n, int count) {
        int most = 0;
        for (int i = 0; i < count; ++i) most = n[i] > most ? n[i] : most;
        const TileChoice free = tuning.choose(prec, nd, n, count);
        const int64_t want = tiles(free, nd, n, count), general = tiles(Tuning::general(prec, nd, most), nd, n, count);
        for (int64_t limit = 1; limit < 400000; limit += 1 + limit / 3) {
            const TileChoice t = tuning.choose(prec, nd, n, count, limit);
            const int64_t k = tiles(t, nd, n, count);
            const bool same = t.tx == free.tx && t.ty == free.ty && t.zchunk == free.zchunk;
            ++all;
            held += want > limit && k <= limit;
            if ((general <= limit && k > limit) || (want <= limit && !same) || t.graph_steps != free.graph_steps) {
                ++bad;
                printf("bad: precision %d, %d-D, n %d (%d samples), limit %lld: %lld tiles\n", prec, nd, n[0], count,
                       (long long)limit, (long long)k);
            }
        }
    };
    for (int prec = 0; prec < 2; ++prec)
        for (int nd = 1; nd <= 3; ++nd) {
            for (int n = 8; n <= 4096; n += 1 + n / 12) check(prec, nd, &n, 1);
            int batch[300];
            for (int i = 0; i < 300; ++i) batch[i] = i % 5 == 4 ? 2 * (20 + i % 60) : 20 + i % 60;
            for (int count : { 2, 7, 40, 300 }) check(prec, nd, batch, count);
            // beyond what a solve takes: the tiling by size
            for (int n : { 4097, 1 << 20, 1 << 30 }) {
                const TileChoice t = tuning.choose(prec, nd, &n, 1), g = Tuning::general(prec, nd, n);
                if (t.tx != g.tx || t.ty != g.ty || t.zchunk != g.zchunk) { ++bad; printf("bad: n %d\n", n); }
            }
        }
    // 2-D double: as many CUs as 16 x 8 tiles, then as 16 x 14 tiles, then two
    // 16 x 8 tiles each; then whichever redoes less
    for (auto [n, ty] : { std::pair(64, 8), { 176, 8 }, { 192, 14 }, { 224, 14 }, { 240, 8 }, { 256, 8 }, { 272, 14 }, { 1024, 14 } })
        if (tuning.choose(1, 2, &n, 1).ty != ty) { ++bad; printf("bad: 2-D double %d\n", n); }
    printf("%ld choices, %ld held to their limit, %ld bad\n", all, held, bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_default_tiling_keeps_to_its_limit(tmp_path):
    src, exe = tmp_path / "tuning.cpp", tmp_path / "tuning"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_1705_04374_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout[-2000:]
    assert " held to their limit, 0 bad" in r.stdout and not r.stdout.startswith("0 choices")
