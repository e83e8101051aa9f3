"""The wide prefill kernel's tiles: the choice and the tile numbering (csrc/lcd_gemm_plan.h, compiled here) on the CPU, every tile shape
on the GPU against the oracle."""
import functools
import random

import numpy as np
import pytest

import synth
import oracle
import paper_2506_12038_amd as lcd
from gemm_plan import HALVES, WHOLE, choices, launches, numbering
from gpu_common import TOL, assert_parity, to_dev


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


# (form, blocks, whether there are columns of one block less) that single calls take
TILES = [(form, blocks, narrower) for form, most in ((0, range(2, 5)), (1, range(2, 5)), (2, range(5, 9))) for blocks in most for narrower in (False, True)]


@functools.lru_cache(None)
def _shapes(bits):
    """Layers with the least work for every tile: rows that end inside a tile, the last token block not full, an even and (halves) an odd number of chunks."""
    rng = random.Random(bits)
    sizes = [(16 * int(2 ** rng.uniform(6, 11)), 256 * int(2 ** rng.uniform(0, 3.5)), int(2 ** rng.uniform(6.1, 11.2))) for _ in range(60000)]
    sizes = [(N, K, M) for N, K, M in sizes if N % 256 and M % 32]
    found = {}
    for (N, K, M), (kernels, *_), (form, blocks, big, columns) in zip(sizes, launches([(bits, M, [(N, K)]) for N, K, M in sizes]),
                                                                        choices([(-1, bits, M, [(N, K)]) for N, K, M in sizes])):
        if kernels[0] in (HALVES, WHOLE):
            key = (form, blocks, big < columns), K // 256 % 2 if form < 2 else 0
            if key not in found or N * K * M < np.prod(found[key]):
                found[key] = N, K, M
    return found


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_layers_for_every_wide_tile(bits):
    assert sorted(_shapes(bits)) == sorted((tile, odd) for tile in TILES for odd in ((0, 1) if tile[0] < 2 else (0,)))


# Sampled rows (the first, the last, tile edges) against the oracle, fp16 activations and INT8 codes; every output written.
@pytest.mark.gpu
@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("bits", [2, 3, 4])
def test_every_wide_tile(bits, tile):
    import torch
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256       # (the plan's)
    for key, (N, K, M) in sorted(_shapes(bits).items()):
        if key[0] != tile:
            continue
        print(bits, key, N, K, M, flush=True)
        layer = synth.make_layer_uniform(N, K, bits, M, seed=N + K + M)
        dev = lcd.lcd_pack_indices(to_dev(layer["idx"]), bits), lcd.lcd_build_lut(to_dev(layer["codebook"]), bits), to_dev(layer["x"]), to_dev(layer["s"])
        rows = np.unique(np.r_[0, 31, 32, 63, 64, 127, 128, 255, 256, N - 17, N - 16, N - 1, np.linspace(0, N - 1, 24).astype(int)])
        args = layer["codebook"][rows], layer["idx"][rows], layer["x"], layer["s"]
        s_q = float(np.float32(np.quantile(np.abs(layer["x"].astype(np.float64) / layer["s"]), 0.99) / 127.0))
        for quantised in (False, True):
            y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
            if quantised:
                lcd.lcd_lut_gemm_q8(*dev, s_q, N, bits, y=y)
            else:
                lcd.lcd_lut_gemm(*dev, N, bits, y=y)
            assert torch.isfinite(y).all(), (key, quantised)
            Y = oracle.quantised_lut_matmul(*args, s_q, bits) if quantised else oracle.lut_matmul(*args, bits)
            assert_parity(y[:, torch.from_numpy(rows).cuda()].cpu().numpy(), Y, 1e-3 if quantised else TOL, (key, quantised))
