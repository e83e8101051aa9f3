"""Workgroups of a grouped decode launch (csrc/lcd_share.h, plain host code): the slowest layer, by the launcher's own cost, is as fast as any
split of the grid makes it, found here by trying every number of workgroups for every layer."""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent

DRIVER = r"""
#include <cstdio>
#include <vector>
#include "lcd_share.h"
using namespace lcd;

static double slowest(const DecodeCost &c, const std::vector<LayerShape> &g, const int *n)
{
    double t = 0.0;
    for (size_t i = 0; i < g.size(); ++i) t = std::max(t, c.time(g[i].bits, g[i].kc, round_up_div(g[i].tiles, n[i])));
    return t;
}
// the smallest T for which the layers' smallest numbers of workgroups fit the grid, every number tried
static double best(const DecodeCost &c, const std::vector<LayerShape> &g, int grid)
{
    std::vector<double> times;
    for (const LayerShape &l : g)
        for (int n = 1; n <= l.tiles && n <= grid; ++n) times.push_back(c.time(l.bits, l.kc, round_up_div(l.tiles, n)));
    std::sort(times.begin(), times.end());
    for (double T : times) {
        int sum = 0;
        for (const LayerShape &l : g) {
            int n = 1;
            while (n <= l.tiles && n <= grid && c.time(l.bits, l.kc, round_up_div(l.tiles, n)) > T) ++n;
            sum += n <= l.tiles ? n : grid + 1;
        }
        if (sum <= grid) return T;
    }
    return -1.0;
}
static int check(const char *name, const DecodeCost &c, const std::vector<LayerShape> &g, int cus)
{
    int tiles = 0, n[kMaxGroup], used = 0;
    for (const LayerShape &l : g) tiles += l.tiles;
    const int grid = std::max((int)g.size(), std::min(cus, tiles));
    share_workgroups(c, g.data(), (int)g.size(), grid, n);
    bool ok = true;
    for (size_t i = 0; i < g.size(); ++i) { used += n[i]; ok = ok && n[i] >= 1 && n[i] <= g[i].tiles; }
    const double got = slowest(c, g, n), want = best(c, g, grid);
    ok = ok && used <= grid && got <= want + 0.02 + 1e-9;     // (the bisection stops there)
    if (!ok) std::printf("%s: grid %d, used %d, %.3f us against %.3f\n", name, grid, used, got, want);
    return ok ? 0 : 1;
}

int main()
{
    int bad = 0;
    unsigned seed = 1u;
    auto rnd = [&](int n) { seed = seed * 1664525u + 1013904223u; return (int)((seed >> 8) % (unsigned)n); };
    auto with_pass = [](DecodeCost c, int pass) { c.pass = pass; return c; };
    struct { const char *name; DecodeCost c; int bits; } kinds[] = {
        {"bucket, 3 bits", bucket_cost(3, 1, false), 3}, {"bucket, 3 bits, codes", bucket_cost(3, 1, true), 3}, {"bucket, 2 bits", bucket_cost(2, 1, false), 2},
        {"bucket, 2 bits, two tokens", bucket_cost(2, 2, false), 2}, {"bucket, 2 bits, two tokens of codes", bucket_cost(2, 2, true), 2},
        {"bucket, 2 bits, three tokens of codes", bucket_cost(2, 3, true), 2}, {"bucket, 2 bits, four tokens of codes", bucket_cost(2, 4, true), 2},
        {"2 bits, codes, passes of three", with_pass(bucket_cost(2, 1, true), 3), 2}, {"2 bits, codes, passes of seven", with_pass(bucket_cost(2, 2, true), 7), 2},
        {"3 bits, codes, passes of five", with_pass(bucket_cost(3, 1, true), 5), 3}, {"tokens, 16", tokens_cost(14, 16, false), 3}, {"tokens, 5, ahead", tokens_cost(14, 5, true), 4}, {"tokens, one pass", tokens_cost(1 << 24, 8, false), 2}, {"narrow, 40", tokens_cost(6, 40, true), 3}};
    for (auto &k : kinds) {
        // row tiles per workgroup around the lengths of the passes: 16 to 22 of them, alone and next to a small layer
        for (int t = 14; t <= 24; ++t) {
            bad += check(k.name, k.c, {{128 * t, 17, k.bits}, {128 * t, 17, k.bits}}, 256);
            bad += check(k.name, k.c, {{200 * t + 3, 43, k.bits}, {56, 17, k.bits}}, 256);
        }
        bad += check(k.name, k.c, {{256, 16, k.bits}, {256, 16, k.bits}, {256, 16, k.bits}}, 256);
        bad += check(k.name, k.c, {{688, 16, k.bits}, {688, 16, k.bits}}, 256);
        bad += check(k.name, k.c, {{256, 16, k.bits}, {256, 16, k.bits}, {256, 16, k.bits}, {256, 16, k.bits}, {688, 16, k.bits}, {688, 16, k.bits}, {256, 43, k.bits}}, 256);
        bad += check(k.name, k.c, {{1, 1, k.bits}, {1, 4, k.bits}, {1, 1, k.bits}}, 2);           // fewer compute units than layers
        for (int r = 0; r < 60; ++r) {
            std::vector<LayerShape> g(1 + rnd(6));
            for (LayerShape &l : g) l = r % 3 == 0 && &l != &g[0] ? g[0] : LayerShape{1 + rnd(r % 2 ? 40 : 2000), 1 + rnd(64), k.c.held ? 2 + rnd(3) : k.bits};
            bad += check(k.name, k.c, g, r % 5 ? 256 : 32);
        }
    }
    // passes: the fewest places and operands, ones and twos only for workgroups of as many row tiles; one chunk per wave: never more than three
    auto pass = [](int bits, int tokens, bool codes, int tiles, int kc) { return kBucketPass[bucket_pass(bucket_rule(bits, tokens, codes), tiles, kc)]; };
    bad += pass(2, 1, true, 2, 16) != 2 || pass(2, 1, true, 4, 16) != 5 || pass(2, 1, true, 6, 16) != 7 || pass(2, 2, true, 8, 32) != 5 || pass(2, 1, true, 9, 32) != 5 ||
           pass(2, 1, false, 6, 32) != 7 || pass(2, 1, false, 15, 20) != 5 || pass(2, 1, false, 21, 32) != 7 || pass(2, 1, false, 22, 16) != 3 || pass(3, 1, true, 12, 20) != 3 ||
           pass(3, 1, false, 8, 32) != 2 || pass(2, 4, true, 14, 32) != 14;
    // layers of different shapes: shares that fill the launch's passes (70B MLP: 21, 21 and 7 row tiles in passes of seven)
    const LayerShape mlp[] = {{1792, 32, 2}, {1792, 32, 2}, {512, 112, 2}};
    for (int tokens = 1; tokens <= 2; ++tokens) {
        int n[kMaxGroup];
        bad += kBucketPass[share_bucket(2, tokens, true, mlp, 3, 256, n)] != 7 || round_up_div(1792, n[0]) != 21 || round_up_div(1792, n[1]) != 21 || round_up_div(512, n[2]) != 7;
    }
    // a workgroup's only pass may have places left over: 7B, 13 and 13 row tiles next to 4; operands of an only chunk are made once: 3072 columns, 8 row tiles in threes
    const LayerShape seven[] = {{256, 16, 3}, {256, 16, 3}, {256, 16, 3}, {256, 16, 3}, {688, 16, 3}, {688, 16, 3}, {256, 43, 3}};
    const LayerShape gqa[] = {{192, 12, 2}, {192, 12, 2}, {64, 12, 2}, {64, 12, 2}, {512, 12, 2}, {512, 12, 2}, {192, 32, 2}};
    int n[kMaxGroup];
    bad += kBucketPass[share_bucket(3, 1, true, seven, 7, 256, n)] != 7 || round_up_div(688, n[4]) != 13 || round_up_div(256, n[6]) != 4;
    bad += kBucketPass[share_bucket(2, 1, false, gqa, 7, 256, n)] != 3 || round_up_div(512, n[4]) != 8;
    std::printf("%d splits worse than the best, or passes not as stated\n", bad);
    return bad ? 1 : 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_shares_are_as_good_as_trying_every_number_of_workgroups(tmp_path):
    (tmp_path / "shares.cpp").write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", f"-I{ROOT / 'include'}", f"-I{ROOT / 'paper_2506_12038_amd' / 'csrc'}",
                           str(tmp_path / "shares.cpp"), "-o", str(tmp_path / "shares")])
    run = subprocess.run([str(tmp_path / "shares")], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout
