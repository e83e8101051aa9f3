"""Helper: the plan of the prefill kernels (csrc/lcd_gemm_plan.h, plain host code) compiled for the tests."""
import functools
import shutil
import subprocess
import tempfile
from pathlib import Path

import pytest

import paper_2506_12038_amd as lcd

CSRC = Path(lcd.__file__).parent / "csrc"
INCLUDE = CSRC.parent.parent / "include"
MAIN = r"""
#include <cstdio>
#include <cstring>
#include "lcd_gemm_plan.h"
using namespace lcd;
static bool read_layers(LayerSize *l, int count)
{
    for (int i = 0; i < count; ++i) if (scanf("%d %d", &l[i].N, &l[i].K) != 2) return false;
    return true;
}
// the wide tiles of layers that a form takes (whole -1: the form of the first layer's rule)
static int choices()
{
    int whole, bits, M, count;
    LayerSize l[16];
    while (scanf("%d %d %d %d", &whole, &bits, &M, &count) == 4) {
        if (!read_layers(l, count)) return 1;
        const WideTiles t = choose_wide(whole < 0 ? whole_takes(M, l[0].N, l[0].K, bits) : whole, l, count, (M + 31) / 32, bits, 256);
        printf("%d %d %d %d\n", t.form, t.blocks, t.big, t.columns);
    }
    return 0;
}
// the numbering: a layer's tiles in either set of columns, then every workgroup's tile
static int tiles()
{
    struct { struct { uint32_t tiles[2]; } p[16]; int count; } batch;
    unsigned blocks;
    while (scanf("%d %u", &batch.count, &blocks) == 2) {
        for (int i = 0; i < batch.count; ++i) if (scanf("%u %u", &batch.p[i].tiles[0], &batch.p[i].tiles[1]) != 2) return 1;
        for (unsigned b = 0; b < blocks; ++b) {
            const WideTileAt at = wide_tile_of(batch, b);
            printf("%d %d %d\n", at.layer, at.second, at.tile);
        }
    }
    return 0;
}
// a call: its layers' kernels, then the launch of the wide layers in halves and of the split layers
static int launches()
{
    int M, bits, count;
    LayerSize l[16];
    while (scanf("%d %d %d", &M, &bits, &count) == 3) {
        LayerSize of[5][16];
        int n[5] = {};
        if (!read_layers(l, count)) return 1;
        for (int i = 0; i < count; ++i) {
            const int k = prefill_kernel(M, l[i].N, l[i].K, bits);
            of[k][n[k]++] = l[i];
            printf("%d ", k);
        }
        const MatrixLaunches p = plan_launches(of[kWideHalves], n[kWideHalves], of[kSplitKernel], n[kSplitKernel], M, bits, 256);
        printf("%d %d %d %d %d %d %d\n", p.together, p.halves.form, p.halves.blocks, p.halves.big, p.halves.columns, p.split ? p.split->pairs : 0, p.split ? p.split->blocks : 0);
    }
    return 0;
}
int main(int, char **argv) { return !strcmp(argv[1], "choices") ? choices() : !strcmp(argv[1], "tiles") ? tiles() : launches(); }
"""
DECODE, NARROW, SPLIT, HALVES, WHOLE = range(5)          # the kernel of a layer


@functools.lru_cache(None)
def _program():
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = Path(tempfile.mkdtemp())
    (d / "plan.cpp").write_text(MAIN)
    subprocess.run(["g++", "-O1", "-std=c++17", f"-I{CSRC}", f"-I{INCLUDE}", str(d / "plan.cpp"), "-o", str(d / "plan")], check=True)
    return d / "plan"


def _run(mode, text):
    out = subprocess.run([str(_program()), mode], input=text, capture_output=True, text=True, check=True).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def choices(cases):
    """(form, blocks, big, columns) of every (whole or -1: as the rule has it, bits, M, [(N, K), ...])."""
    return _run("choices", "\n".join(f"{w} {b} {M} {len(ls)} " + " ".join(f"{n} {k}" for n, k in ls) for w, b, M, ls in cases))


def numbering(tiles, blocks):
    """(layer, second, tile) of every one of `blocks` workgroups; tiles: a layer's in either set of columns."""
    return _run("tiles", f"{len(tiles)} {blocks}\n" + "\n".join(f"{a} {b}" for a, b in tiles))


def launches(cases):
    """(the layers' kernels, together, (form, blocks, big, columns), (pairs, blocks)) of every (bits, M, [(N, K), ...])."""
    out = _run("launches", "\n".join(f"{M} {b} {len(ls)} " + " ".join(f"{n} {k}" for n, k in ls) for b, M, ls in cases))
    return [(r[:-7], bool(r[-7]), r[-6:-2], r[-2:]) for r in out]
