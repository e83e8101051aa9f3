"""The wide prefill kernel's tiles: the choice and the tile numbering (csrc/lcd_gemm_plan.h, compiled here) on the CPU, every tile shape
on the GPU against the oracle."""
import functools
import random

import numpy as np
import pytest

import synth
import oracle
import paper_2506_12038_amd as lcd
from gemm_plan import choices, numbering
from gpu_common import assert_parity, to_dev


def _case(rng):
    layers = [(16 * rng.randint(1, 2000), 256 * rng.randint(1, 112)) for _ in range(rng.choice([1, 1, 2, 3, 16]))]
    return rng.choice([0, 1]), rng.choice([2, 3, 4]), int(2 ** rng.uniform(0, 13)), layers


def test_columns_hold_every_block_once():
    rng = random.Random(7)
    cases = [_case(rng) for _ in range(2000)]
    for (whole, bits, M, layers), (form, blocks, big, columns) in zip(cases, choices(cases)):
        token_blocks = -(-M // 32)
        if whole and token_blocks < 5:
            assert columns == 0           # (no such tile: the rule never asks for one)
            continue
        assert form == 2 if whole else form in (0, 1)
        assert (5 <= blocks <= 8) if whole else (1 <= blocks <= 4)
        assert 1 <= big <= columns and big * blocks + (columns - big) * (blocks - 1) == token_blocks


def test_whole_layers_have_whole_tiles():
    rng = random.Random(8)
    cases = [(-1, b, M, ls[:1]) for _, b, M, ls in (_case(rng) for _ in range(2000))]
    assert all(columns > 0 for _, _, _, columns in choices(cases))


@pytest.mark.parametrize("seed", range(20))
def test_every_tile_has_one_workgroup(seed):
    rng = random.Random(seed)
    tiles = [[rng.choice([0, rng.randint(1, 20), rng.randint(1, 400)]) for _ in range(2)] for _ in range(rng.choice([1, 1, 2, 3, 7, 16]))]
    queue = -(-sum(map(sum, tiles)) // 8)        # the launch: as many workgroups on every XCD
    got = numbering(tiles, 8 * queue)
    assert len(got) == 8 * queue
    assert sorted(t for t in got if t[0] >= 0) == [(i, s, t) for i, sets in enumerate(tiles) for s in (0, 1) for t in range(sets[s])]
    # an XCD's workgroups go through the wider columns of all layers first, a layer's tiles in rising order
    for xcd in range(8):
        own = [(s, i, t) for i, s, t in got[xcd::8] if i >= 0]
        assert own == sorted(own)


@functools.lru_cache(None)
def _shapes(bits):
    """A layer for every (form, blocks, whether there are columns of one block less) that a single call takes."""
    sizes = [(N, K, M) for K in (512, 768) for N in (4112, 8208, 16400, 20496) for M in range(130, 2049, 61) if -(-N // 64) * -(-M // 128) > 256]
    found = {}
    for (N, K, M), (form, blocks, big, columns) in zip(sizes, choices([(-1, bits, M, [(N, K)]) for N, K, M in sizes])):
        found.setdefault((form, blocks, big < columns), (N, K, M))
    return found


# Rows that end inside a tile (N = 16 more than a multiple of 256), two and three chunks of K, the last token block not full, columns of
# one width and of two.  Sampled rows (the first, the last, tile edges) against the oracle.
@pytest.mark.gpu
@pytest.mark.parametrize("bits", [2, 3, 4])
def test_every_wide_tile(bits):
    import torch
    found = _shapes(bits)
    assert {f for f, _, _ in found} == {0, 1, 2}
    for key, (N, K, M) in sorted(found.items()):
        layer = synth.make_layer_uniform(N, K, bits, M, seed=N + K + M)
        packed, lut = lcd.lcd_pack_indices(to_dev(layer["idx"]), bits), lcd.lcd_build_lut(to_dev(layer["codebook"]), bits)
        y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
        lcd.lcd_lut_gemm(packed, lut, to_dev(layer["x"]), to_dev(layer["s"]), N, bits, y=y)
        y = y.cpu().numpy()
        assert np.isfinite(y).all(), key
        rows = np.unique(np.r_[0, 31, 32, 63, 64, 127, 128, 255, 256, N - 17, N - 16, N - 1, np.linspace(0, N - 1, 24).astype(int)])
        assert_parity(y[:, rows], oracle.lut_matmul(layer["codebook"][rows], layer["idx"][rows], layer["x"], layer["s"], bits))
