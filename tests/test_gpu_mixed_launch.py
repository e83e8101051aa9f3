"""The prefill launch that takes wide and split tiles together: every variant of it that calls take (split tiles of 96 and 128 tokens; wide tiles
of 128 and 256 rows, of 3 and 4 blocks, columns of one width and of two) at every index width, fp16 activations and INT8 codes, against the oracle
and bit for bit against the layers' own calls.  The groups are searched with the plan the library is built from (csrc/lcd_gemm_plan.h)."""
import functools
import random

import numpy as np
import pytest

import synth
import oracle
import paper_2506_12038_amd as lcd
from paper_2506_12038_amd.binding import GemmGroup
from gemm_plan import HALVES, SPLIT, launches
from gpu_common import TOL, assert_parity, to_dev


def _variants(bits):
    """(split blocks, wide form, wide blocks, columns of one block less next to them) that calls take.  Where every wide tile has 4 blocks, split tiles of 4 have
    the least work; at 4 bits, whose split tiles of 3 blocks cost nearly as much, wherever some have."""
    return [(s, f, b, n) for s in (3, 4) for f in (0, 1) for b, n in ((3, False), (4, False), (4, True)) if not (s == 3 and b == 4 and (not n or bits == 4))]


@functools.lru_cache(None)
def _groups(bits):
    """The group with the least work for every variant.  Rows that end inside a wide and a split tile, a last token block that is not full, an odd and
    an even number of chunks."""
    rng, cases = random.Random(bits), []
    for _ in range(30000):
        wide = [(16 * rng.randint(129, 1400), 256 * rng.choice([1, 2, 3, 5])) for _ in range(rng.choice([1, 1, 2]))]
        split = [(16 * rng.randint(1, 130), 256 * rng.choice([1, 2, 9])) for _ in range(rng.choice([1, 2]))]
        cases.append((bits, rng.randint(97, 700), rng.sample(wide + split, len(wide) + len(split))))
    found = {}
    for (_, M, layers), (kernels, together, (form, blocks, big, columns), split) in zip(cases, launches(cases)):
        odd = M % 32 and any(N % 256 for (N, _), k in zip(layers, kernels) if k == HALVES) and any(N % 64 for (N, _), k in zip(layers, kernels) if k == SPLIT)
        if together and set(kernels) == {HALVES, SPLIT} and odd:
            key, work = (split[1], form, blocks, big < columns), M * sum(N * K for N, K in layers)
            if key not in found or work < found[key][0]:
                found[key] = work, M, layers
    return {key: (M, layers) for key, (_, M, layers) in found.items()}


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_groups_for_every_variant(bits):
    assert sorted(_groups(bits)) == sorted(_variants(bits))


@pytest.mark.gpu
@pytest.mark.parametrize("bits,variant", [(bits, v) for bits in (2, 3, 4) for v in _variants(bits)])
def test_every_variant(bits, variant):
    import torch
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256       # (the plan's)
    M, shapes = _groups(bits)[variant]
    print(bits, variant, M, shapes, flush=True)
    layers = [synth.make_layer_uniform(N, K, bits, M, seed=N + K + M) for N, K in shapes]
    dev = [(lcd.lcd_pack_indices(to_dev(l["idx"]), bits), lcd.lcd_build_lut(to_dev(l["codebook"]), bits), to_dev(l["x"]), to_dev(l["s"])) for l in layers]
    for quantised in (False, True):
        steps = [float(np.float32(np.quantile(np.abs(l["x"].astype(np.float64) / l["s"]), 0.99) / 127.0)) for l in layers]
        y = [torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for N, _ in shapes]
        problems = [(*d, o, N) for d, o, (N, _) in zip(dev, y, shapes)]
        GemmGroup(problems, bits, s_q=steps if quantised else None)()
        for layer, d, o, s_q, (N, K) in zip(layers, dev, y, steps, shapes):
            single = lcd.lcd_lut_gemm_q8(*d, s_q, N, bits) if quantised else lcd.lcd_lut_gemm(*d, N, bits)
            assert torch.equal(o, single), (N, K, quantised)
            rows = np.unique(np.r_[0, N - 1, np.linspace(0, N - 1, 32).astype(int)])
            args = layer["codebook"][rows], layer["idx"][rows], layer["x"], layer["s"]
            Y = oracle.quantised_lut_matmul(*args, s_q, bits) if quantised else oracle.lut_matmul(*args, bits)
            assert_parity(o.cpu().numpy()[:, rows], Y, 1e-3 if quantised else TOL, (N, K, quantised))
