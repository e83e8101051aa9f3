"""GPU: batched decode (2 <= M <= 16) and prefill (lcd_lut_gemm) against the fp64 CPU oracle."""
import numpy as np
import pytest

import oracle
import synth
import paper_2506_12038_amd as lcd
from gemm_plan import HALVES, NARROW, SPLIT, WHOLE, choices, launches
from gpu_common import TOL, assert_parity, check_layer, config_layers, run_hip, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("M", [2, 3, 8, 16])
@pytest.mark.parametrize("shape", [(16, 256), (48, 768), (80, 2304), (64, 11008), (32, 28672), (96, 5120), (48, 6656), (32, 13824), (8208, 1280)])
def test_gemv_batched_small(bits, M, shape):
    N, K = shape
    layer = synth.make_layer(2, 0, N, K, bits, M, seed_offset=N + K + M)
    check_layer(layer, bits, "gemv")


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("M", [16, 17, 31, 32])
@pytest.mark.parametrize("shape", [(16, 256), (48, 2304), (16 * 700, 512), (16 * 1800, 256)])
def test_gemm_token_block_edges(bits, M, shape):
    # the tokens kernel behind lcd_lut_gemm: one and two 16-token blocks, fewer chunks than waves, a short last round of
    # chunks, and 1, 2, 3 and 7-8 row tiles per workgroup (one and several passes over K)
    N, K = shape
    check_layer(synth.make_layer_uniform(N, K, bits, M, seed=N + K + M), bits, "gemm")


# The tokens kernel with several row tiles per workgroup: fewer tiles than its ring of packed words has slots in a
# pass (the last of two), one tile either side of the smaller variants, of what it holds (14) and of two full passes; up to K = 4096, where every
# wave's operands stay, passes of three tiles that fill the partial tiles' places (six) or not; activations
# smoothed in the kernel, for 4, 8 or 16 tokens, and (INT8 codes, 16 tokens) transformed ahead.  Most workgroups have `tiles` row tiles, a few one less.
# (One token: 4 bits only, the other widths take the bucket kernel.)
@pytest.mark.parametrize("bits,M,quantised", [(4, 1, False)] + [(b, M, q) for b in (2, 3, 4) for M, q in ((3, False), (6, False), (16, False), (16, True))])
@pytest.mark.parametrize("tiles,K", [(2, 4352), (3, 4096), (3, 8704), (4, 2304), (5, 2304), (5, 4352), (6, 4096), (7, 4352), (8, 512), (13, 2304), (14, 4352), (15, 2304), (15, 4352),
                                     (28, 1280), (29, 2304), (29, 4352)])
def test_gemv_many_row_tiles_per_workgroup(bits, tiles, K, M, quantised):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rows = cus * 16                                   # one tile per workgroup
    N = tiles * rows - 48
    g = torch.Generator(device="cuda")
    g.manual_seed(tiles * K + M)
    packed = torch.randint(0, 256, (lcd.lcd_packed_bytes(N, K, bits),), dtype=torch.uint8, device="cuda", generator=g)
    codebook = (torch.randn((N, 1 << bits), device="cuda", generator=g) * 0.02).half()
    x = torch.randn((M, K), device="cuda", generator=g).half()
    s = torch.rand((K,), device="cuda", generator=g) + 0.5
    s_q = 0.03
    if quantised:
        call = lambda p, l, n, **kw: lcd.lcd_lut_gemv_q8(p, l, x, s, s_q, n, bits, **kw)
    else:
        call = lambda p, l, n, **kw: lcd.lcd_lut_gemv(p, l, x, s, n, bits, **kw)
    y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
    call(packed, lcd.lcd_build_lut(codebook, bits), N, y=y)
    for first in range(0, N, rows):                   # the same rows in calls of one tile per workgroup: the same bits
        n = min(rows, N - first)
        part = packed[lcd.lcd_packed_bytes(first, K, bits) if first else 0:][:lcd.lcd_packed_bytes(n, K, bits)].clone()
        cb = codebook[first:first + n].contiguous()
        assert torch.equal(y[:, first:first + n], call(part, lcd.lcd_build_lut(cb, bits), n)), first
    idx = lcd.lcd_unpack_indices(part, n, K, bits).cpu().numpy()
    args = cb.cpu().numpy(), idx, x.cpu().numpy(), s.cpu().numpy()
    Y = oracle.quantised_lut_matmul(*args, s_q, bits) if quantised else oracle.lut_matmul(*args, bits)
    assert_parity(y[:, first:].cpu().numpy(), Y, 1e-3 if quantised else TOL)


# the same for the forms chosen to stay clear of spills, 9 to 16 tokens made in the kernel: 2 bits, 12 row tiles a pass where 14 need as many, row
# tables in LDS beyond, four and five tiles on forms of their own, six with a ring; 4 bits, two row tiles: 8 waves up to 12 chunks and beyond 16, resident between
@pytest.mark.parametrize("bits,tiles,K", [(2, 12, 4352), (2, 13, 4352), (2, 24, 4352), (2, 25, 4352), (2, 4, 4352), (2, 4, 6400), (2, 5, 4352), (2, 5, 6400), (2, 6, 4352), (2, 6, 6400), (2, 5, 7168), (4, 2, 3072), (4, 2, 3328), (4, 2, 4096)])
@pytest.mark.parametrize("M", [9, 16])
def test_gemv_forms_clear_of_spills(bits, tiles, K, M):
    test_gemv_many_row_tiles_per_workgroup(bits, tiles, K, M, False)


# the bucket kernel's passes of five and seven row tiles: full, one tile short and one over
@pytest.mark.parametrize("bits,M,quantised", [(2, 1, True), (2, 2, True), (2, 1, False), (3, 1, True)])
@pytest.mark.parametrize("tiles,K", [(4, 2304), (5, 4352), (6, 4352), (8, 4352), (9, 2304), (10, 4352), (15, 4352), (16, 4608)])
def test_bucket_passes(bits, M, quantised, tiles, K):
    test_gemv_many_row_tiles_per_workgroup(bits, tiles, K, M, quantised)


# the split kernel behind lcd_lut_gemm: one token either side of a tile, rows that fill half a pair, fewer 128-column units than
# waves (K = 256), units that do not divide by the waves (K = 1280, 2304); and layers around the ends of its range, which the narrow (few
# tokens) or the wide kernel takes (at 2 bits, whose range is shorter, some that are its own at 3 and 4)
@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("shape", [(48, 1280, 33), (48, 1280, 64), (48, 2304, 33), (48, 2304, 64), (5136, 256, 65), (1040, 512, 300), (5136, 256, 34), (5136, 1280, 65), (5136, 256, 97), (5136, 256, 200),
                                   (5136, 2304, 300), (8016, 2304, 129), (4096, 4096, 17), (4112, 4096, 32), (28800, 256, 128), (28800, 256, 257), (16384, 256, 128), (16400, 256, 128),
                                   (32768, 256, 64), (32784, 256, 64), (10912, 512, 192), (10928, 512, 192)])
def test_gemm_split_tile_edges(bits, shape):
    N, K, M = shape
    check_layer(synth.make_layer_uniform(N, K, bits, M, seed=N + K + M), bits, "gemm")


# the narrow kernel: one token either side of a block of 16, every number of blocks; row tiles per workgroup up to, at and past what a
# variant holds (6, 4, 3) and in more than one pass; fewer chunks than waves, one and several per wave
@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("N,K,M", [(4096, 4096, 17), (4096, 4352, 32), (48, 1280, 33), (4112, 256, 33), (4112, 2304, 48), (2064, 512, 49), (12288, 256, 64), (20496, 512, 64), (16400, 2304, 50),
                                   (24592, 256, 47), (32800, 512, 20), (6144, 2304, 65), (6160, 256, 80), (12288, 512, 81), (8208, 4352, 96)])
def test_gemm_narrow_kernel_edges(bits, N, K, M):
    assert launches([(bits, M, [(N, K)])])[0][0] == (NARROW,)
    check_layer(synth.make_layer_uniform(N, K, bits, M, seed=N + K + M), bits, "gemm")


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("M", [24, 40, 64, 90])
def test_narrow_kernel_grouped_and_quantised(bits, M):
    # layers on the narrow, the split and (small ones, up to 32 tokens) the tokens kernel in one call, inputs shared or not: the bits of single calls
    import torch
    from paper_2506_12038_amd.binding import GemmGroup
    g = torch.Generator(device="cuda")
    g.manual_seed(M + bits)
    for q8 in (False, True):
        problems, steps = [], []
        shared = {}
        for i, (N, K) in enumerate([(6160, 2304), (64, 512), (8208, 2304), (4096, 5120), (6144, 4096)]):
            if K not in shared or i == 2:
                shared[K] = (torch.randn((M, K), device="cuda", generator=g).half(), torch.rand((K,), device="cuda", generator=g) + 0.5)
            packed = torch.randint(0, 256, (lcd.lcd_packed_bytes(N, K, bits),), dtype=torch.uint8, device="cuda", generator=g)
            lut = lcd.lcd_build_lut((torch.randn((N, 1 << bits), device="cuda", generator=g) * 0.02).half(), bits)
            problems.append((packed, lut, *shared[K], torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda"), N))
            steps.append(0.03)
        GemmGroup(problems, bits, s_q=steps if q8 else None)()
        for packed, lut, x, s, y, N in problems:
            single = lcd.lcd_lut_gemm_q8(packed, lut, x, s, 0.03, N, bits) if q8 else lcd.lcd_lut_gemm(packed, lut, x, s, N, bits)
            assert torch.equal(y, single), (N, q8)


# every tile of the split kernel at every width, with an uneven number of 128-column units per wave (K = 2304: 18 units on 8
# waves; K = 1792, for 64 x 32 at 4 bits, which longer rows do not take: 14), so that a wave refills its ring, its packed words
# and its operands across units; a last row tile in half a pair, a last token block that is not full
@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("tile", [(1, 1), (1, 2), (2, 1), (2, 2), (2, 3), (2, 4)])
def test_gemm_every_split_tile(bits, tile):
    rows = [48 + 928 * i for i in range(37)] + [2704]
    sizes = [(N, K, M) for K in (2304, 1792) for M in (45, 77, 109, 141, 173, 237) for N in rows]
    plans = launches([(bits, M, [(N, K)]) for N, K, M in sizes])
    found = [size for size, (kernels, _, _, split) in zip(sizes, plans) if kernels == (SPLIT,) and split == tile]
    assert found
    N, K, M = found[0]
    check_layer(synth.make_layer_uniform(N, K, bits, M, seed=N + K + M), bits, "gemm")


# the wide kernel on many token blocks: rows that end in a tile's first rows, in its middle and with it, a last token block of 24, 32 and one token
@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("shape", [(4112, 256, 2040), (4240, 512, 2048), (8336, 512, 1025), (6144, 256, 1985)])
def test_gemm_wide_long_prompts(bits, shape):
    N, K, M = shape
    check_layer(synth.make_layer_uniform(N, K, bits, M, seed=N + K + M), bits, "gemm")


# wide layers that take other tiles in a group than on their own, in halves and whole: the same bits
@pytest.mark.parametrize("M,shapes,kernel", [(387, [(9424, 768), (4784, 768)], HALVES), (579, [(10400, 768), (9888, 768)], WHOLE)])
def test_gemm_tiles_that_depend_on_the_group(M, shapes, kernel):
    assert launches([(3, M, shapes)])[0][0] == (kernel, kernel)
    together, *alone = choices([(int(kernel == WHOLE), 3, M, layers) for layers in (shapes, shapes[:1], shapes[1:])])
    assert all(tile[:2] != together[:2] for tile in alone)
    _check_grouped_prefill(3, M, shapes)


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("M", [1, 2, 3, 20, 40])
def test_gemm_infinite_activation_stays_in_its_token(bits, M):
    # one infinite activation: its token's outputs are the infinity of the centroid's sign (as plain arithmetic
    # gives), the others are what they are without it -- on every kernel that takes few tokens
    N, K = 80, 1280
    layer = synth.make_layer_uniform(N, K, bits, M, seed=bits + M)
    Y = oracle.lut_matmul(layer["codebook"], layer["idx"], layer["x"], layer["s"], bits)
    layer["x"] = layer["x"].copy()
    layer["x"][M - 1, 700] = np.inf
    y = run_hip(layer, bits, "gemm")
    centroid = layer["codebook"][np.arange(N), layer["idx"][:, 700]].astype(np.float64)
    assert np.all(centroid != 0)
    assert np.array_equal(y[M - 1], np.copysign(np.inf, centroid))
    if M > 1:
        assert_parity(y[:M - 1], Y[:M - 1])


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("M", [1, 5, 64, 130, 257])
@pytest.mark.parametrize("shape", [(16, 256), (48, 768), (272, 1024), (1040, 512)])
def test_gemm_small(bits, M, shape):
    N, K = shape
    layer = synth.make_layer(3, 0, N, K, bits, M, seed_offset=N + K + M)
    check_layer(layer, bits, "gemm")


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("entry", ["gemv", "gemm"])
def test_batched_one_hot_rows_are_exact(bits, entry):
    # token m has x = e_{k_m}, s = 1: y[m][n] = C[n][idx[n][k_m]] exactly
    import torch
    N, K, M = 32, 512, 16
    layer = synth.make_layer(0, 0, N, K, bits, 1, seed_offset=9)
    packed = lcd.lcd_pack_indices(to_dev(layer["idx"]), bits)
    lut = lcd.lcd_build_lut(to_dev(layer["codebook"]), bits)
    s = torch.ones(K, dtype=torch.float32, device="cuda")
    fn = lcd.lcd_lut_gemv if entry == "gemv" else lcd.lcd_lut_gemm
    for base in range(0, 256, 16):
        ks = [base + m for m in range(M)]
        x = torch.zeros((M, K), dtype=torch.float16, device="cuda")
        for m, k in enumerate(ks):
            x[m, k] = 1.0
        y = fn(packed, lut, x, s, N, bits).cpu().numpy()
        for m, k in enumerate(ks):
            assert np.array_equal(y[m], layer["codebook"][np.arange(N), layer["idx"][:, k]]), (m, k)


def _grouped_outputs(cfg_index, M, entry):
    """All matrices of a config through ONE grouped call (the launch configuration bench.py times);
    returns [(spec, layer, y)] with y as numpy.  Outputs start as NaN."""
    import torch
    config = synth.get_config(cfg_index)
    problems, keep = [], []
    for mid, spec, layer in config_layers(cfg_index, M, distinct_shapes_only=False):
        packed = lcd.lcd_pack_indices(to_dev(layer["idx"]), config.bits)
        lut = lcd.lcd_build_lut(to_dev(layer["codebook"]), config.bits)
        y = torch.full((M, spec.N), float("nan"), dtype=torch.float16, device="cuda")
        problems.append((packed, lut, to_dev(layer["x"]), to_dev(layer["s"]), y, spec.N))
        keep.append((spec, layer))
    (lcd.lcd_lut_gemv_grouped if entry == "gemv" else lcd.lcd_lut_gemm_grouped)(problems, config.bits)
    torch.cuda.synchronize()
    return [(spec, layer, p[4].cpu().numpy()) for (spec, layer), p in zip(keep, problems)]


def _check_every_output(cfg_index, M):
    """Every output of every matrix of a decode config against the oracle: the grouped call over the
    whole set, and the single call on the first matrix of each shape."""
    bits = synth.get_config(cfg_index).bits
    seen = set()
    for spec, layer, y in _grouped_outputs(cfg_index, M, "gemv"):
        Y = oracle.lut_matmul(layer["codebook"], layer["idx"], layer["x"], layer["s"], bits)
        assert_parity(y, Y, what=("grouped call", cfg_index, M, spec))
        if (spec.N, spec.K) not in seen:
            seen.add((spec.N, spec.K))
            assert_parity(run_hip(layer, bits, "gemv"), Y, what=("single call", cfg_index, M, spec))


def test_config2_batched_decode_full_size_every_output():
    _check_every_output(2, 16)


def test_config2_shapes_two_tokens_full_size_every_output():
    # two tokens at 2 bits run on the sparse-matrix-core kernel (one pass per token)
    _check_every_output(2, 2)


@pytest.mark.parametrize("M", [1, 3, 4])
def test_config2_shapes_int8_codes_full_size_every_output(M):
    # 2 bits with the INT8 codes of Sec. 4.1: up to four tokens run on the sparse-matrix-core kernel with
    # int8 operands.  One grouped call over the whole set, every output against the quantised oracle.
    import torch
    from paper_2506_12038_amd.binding import GemvGroup
    config = synth.get_config(2)
    problems, keep, steps = [], [], []
    for mid, spec, layer in config_layers(2, M, distinct_shapes_only=False):
        packed = lcd.lcd_pack_indices(to_dev(layer["idx"]), config.bits)
        lut = lcd.lcd_build_lut(to_dev(layer["codebook"]), config.bits)
        y = torch.full((M, spec.N), float("nan"), dtype=torch.float16, device="cuda")
        problems.append((packed, lut, to_dev(layer["x"]), to_dev(layer["s"]), y, spec.N))
        steps.append(float(np.float32(np.quantile(np.abs(layer["x"].astype(np.float64) / layer["s"]), 0.99) / 127.0)))
        keep.append((spec, layer))
    GemvGroup(problems, config.bits, s_q=steps)()
    torch.cuda.synchronize()
    for (spec, layer), p, s_q in zip(keep, problems, steps):
        got = p[4].cpu().numpy()
        assert np.all(np.isfinite(got.astype(np.float32))), spec
        Y = oracle.quantised_lut_matmul(layer["codebook"], layer["idx"], layer["x"], layer["s"], s_q, config.bits)
        err = oracle.parity_errors(got, Y)
        assert err["max_rel_floored"] <= 1e-3, (spec, M, err)


@pytest.mark.parametrize("M", [1, 8])
def test_config4_70b_mlp_full_size_every_output(M):
    _check_every_output(4, M)


def _check_prefill_sample(spec, layer, y, bits, mid, M):
    """Prefill outputs are too many for the oracle (2048 tokens): every row for 8 sampled tokens and
    every token for 96 sampled rows, both with the first and the last one; finite everywhere."""
    assert np.all(np.isfinite(y.astype(np.float32))), spec
    rng = np.random.default_rng(99 + mid)
    ms = np.sort(rng.choice(M, size=8, replace=False)); ms[0] = 0; ms[-1] = M - 1
    Y = oracle.lut_matmul(layer["codebook"], layer["idx"], layer["x"][ms], layer["s"], bits)
    assert_parity(y[ms], Y, what=("all rows of sampled tokens", spec))
    rs = np.sort(rng.choice(spec.N, size=96, replace=False)); rs[0] = 0; rs[-1] = spec.N - 1
    Y = oracle.lut_matmul(layer["codebook"][rs], layer["idx"][rs], layer["x"], layer["s"], bits)
    # rms over the sampled rows stands in for the row rms (rows are i.i.d. by construction)
    assert_parity(y[:, rs], Y, what=("all tokens of sampled rows", spec))


def test_config3_prefill_full_size_single_calls():
    bits, M = synth.get_config(3).bits, 2048
    for mid, spec, layer in config_layers(3, M, distinct_shapes_only=True):
        _check_prefill_sample(spec, layer, run_hip(layer, bits, "gemm"), bits, mid, M)


def test_config3_prefill_full_size_grouped_call():
    bits, M = synth.get_config(3).bits, 2048
    for mid, (spec, layer, y) in enumerate(_grouped_outputs(3, M, "gemm")):
        _check_prefill_sample(spec, layer, y, bits, mid, M)


@pytest.mark.parametrize("bits,ncent", [(3, 5), (3, 6), (4, 10), (4, 13)])
@pytest.mark.parametrize("M,entry", [(1, "gemv"), (6, "gemv"), (70, "gemm")])
def test_codebooks_with_fewer_centroids_than_the_container_holds(bits, ncent, M, entry):
    # centroid counts that are no power of two (the paper's per-layer counts: 5, 6, 10, ...) live in the
    # next container; the codes above the count are never used and their table entries are zero
    N, K = 80, 1280
    layer = synth.make_layer(1, 3, N, K, bits, M, seed_offset=bits + ncent + M)
    layer["idx"] = (layer["idx"] % ncent).astype(np.uint8)
    layer["codebook"] = layer["codebook"].copy()
    layer["codebook"][:, ncent:] = 0
    assert int(layer["idx"].max()) == ncent - 1
    check_layer(layer, bits, entry)


@pytest.mark.parametrize("bits,M", [(2, 200), (3, 64), (3, 300), (4, 129)])
def test_grouped_prefill_matches_single_calls_and_oracle(bits, M):
    # several layers of different N and K in one pair of launches: the same bits as lcd_lut_gemm layer by layer
    _check_grouped_prefill(bits, M, [(272, 1024), (1040, 512), (48, 2816), (4112, 256), (16, 4352)])


# layers of one call on different kernels: decode and narrow; split and wide, in a launch of their own (129 tokens: five blocks have no tiles for both) and in
# one (every variant of that launch: test_gpu_mixed_launch.py), layers that end inside a tile of either kind
@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("M,shapes", [(20, [(64, 512), (8192, 2048), (4096, 4096), (48, 2816)]),
                                      (129, [(16912, 256), (256, 512), (17040, 256), (4112, 256)]),
                                      (110, [(34320, 256), (48, 2304), (1040, 512)]),
                                      (110, [(36624, 256), (1040, 2304), (16, 256)]),
                                      (257, [(272, 1280), (12304, 512), (16, 4352)]),
                                      (513, [(12816, 256), (80, 2304), (4112, 256), (13072, 256)])])
def test_grouped_prefill_with_layers_on_different_kernels(bits, M, shapes):
    _check_grouped_prefill(bits, M, shapes)


def _check_grouped_prefill(bits, M, shapes):
    import torch
    problems, layers, singles = [], [], []
    for i, (N, K) in enumerate(shapes):
        layer = synth.make_layer(3, i, N, K, bits, M, seed_offset=5 * i + bits + M)
        packed = lcd.lcd_pack_indices(to_dev(layer["idx"]), bits)
        lut = lcd.lcd_build_lut(to_dev(layer["codebook"]), bits)
        x, s = to_dev(layer["x"]), to_dev(layer["s"])
        y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
        problems.append((packed, lut, x, s, y, N))
        layers.append(layer)
        singles.append(lcd.lcd_lut_gemm(packed, lut, x, s, N, bits))
    lcd.lcd_lut_gemm_grouped(problems, bits)
    torch.cuda.synchronize()
    for (packed, lut, x, s, y, N), layer, single in zip(problems, layers, singles):
        assert torch.equal(y, single)
        Y = oracle.lut_matmul(layer["codebook"], layer["idx"], layer["x"], layer["s"], bits)
        assert oracle.parity_errors(y.cpu().numpy(), Y)["max_rel_floored"] <= TOL


def test_grouped_prefill_config3_sampled_and_replayed_from_a_hip_graph():
    # the launch configuration bench.py times for the prefill config: the whole 7B set in one grouped
    # call, captured once and replayed; sampled rows against the oracle, every replay against the eager call
    import torch
    from paper_2506_12038_amd.binding import GemmGroup
    config = synth.get_config(3)
    M = 256
    problems, samples = [], []
    for mid, spec in config.matrices():
        layer = synth.make_layer(3, mid, spec.N, spec.K, config.bits, M)
        packed = lcd.lcd_pack_indices(to_dev(layer["idx"]), config.bits)
        lut = lcd.lcd_build_lut(to_dev(layer["codebook"]), config.bits)
        y = torch.zeros((M, spec.N), dtype=torch.float16, device="cuda")
        problems.append((packed, lut, to_dev(layer["x"]), to_dev(layer["s"]), y, spec.N))
        rs = np.sort(np.random.default_rng(mid).choice(spec.N, size=64, replace=False))
        rs[0] = 0; rs[-1] = spec.N - 1
        samples.append((rs, oracle.lut_matmul(layer["codebook"][rs], layer["idx"][rs], layer["x"], layer["s"], config.bits)))
        del layer
    group = GemmGroup(problems, config.bits)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        group(stream)
    torch.cuda.synchronize()
    eager = [p[4].clone() for p in problems]
    for (rs, Y), e in zip(samples, eager):
        assert oracle.parity_errors(e.cpu().numpy()[:, rs], Y)["max_rel_floored"] <= TOL
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        group(stream)
    for rep in range(3):
        for p in problems:
            p[4].fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            graph.replay()
        torch.cuda.synchronize()
        for p, e in zip(problems, eager):
            assert torch.equal(p[4], e), rep


@pytest.mark.parametrize("count", [1, 16])
def test_grouped_prefill_smallest_and_largest_group(count):
    # one layer (the grouped call degenerates to lcd_lut_gemm) and the largest group the entry point takes
    import torch
    bits, M = 3, 70
    problems, singles = [], []
    for i in range(count):
        N, K = 16 * (1 + i % 5), 256 * (1 + (3 * i) % 4)
        layer = synth.make_layer(3, i, N, K, bits, M, seed_offset=11 * i + count)
        packed = lcd.lcd_pack_indices(to_dev(layer["idx"]), bits)
        lut = lcd.lcd_build_lut(to_dev(layer["codebook"]), bits)
        x, s = to_dev(layer["x"]), to_dev(layer["s"])
        y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
        problems.append((packed, lut, x, s, y, N))
        singles.append(lcd.lcd_lut_gemm(packed, lut, x, s, N, bits))
        Y = oracle.lut_matmul(layer["codebook"], layer["idx"], layer["x"], layer["s"], bits)
        assert oracle.parity_errors(singles[-1].cpu().numpy(), Y)["max_rel_floored"] <= TOL
    lcd.lcd_lut_gemm_grouped(problems, bits)
    torch.cuda.synchronize()
    for p, single in zip(problems, singles):
        assert torch.equal(p[4], single)



class _WatchedWorkspace:
    """A workspace filled with a pattern: whether a call has written into it."""

    def __init__(self, nbytes):
        import torch
        self.tensor = torch.full((max(nbytes, 256),), 0xA5, dtype=torch.uint8, device="cuda")

    def written(self):
        return bool((self.tensor != 0xA5).any())


# ahead: of the single call and of the group of two (256 compute units: 257 row tiles or more, K = 8192; 769 or more, K = 6656, 2 bits 7424)
@pytest.mark.parametrize("bits,M,N,K,ahead", [(2, 9, 4112, 8192, (True, True)), (4, 16, 4112, 8192, (True, True)), (3, 9, 4112, 7936, (False, False)), (3, 10, 12304, 6656, (True, True)),
                                              (2, 16, 12288, 6656, (False, False)), (3, 16, 12288, 6656, (False, True)), (2, 9, 12304, 7168, (False, False)), (2, 9, 12288, 7424, (False, True)),
                                              (4, 11, 4096, 8448, (False, True)), (3, 8, 4112, 8192, (False, False))])
def test_gemv_smoothed_in_and_ahead_of_the_product(bits, M, N, K, ahead):
    # either side of the lines for fp16 activations of 9 to 16 tokens (row tiles per compute unit, columns): whole calls against calls
    # of up to 8 tokens, which smooth inside the kernel, bit for bit (the order of the additions depends on K alone), single and two layers in one launch.
    # Which side a call is on shows in its workspace: smoothed activations are written there.
    import torch
    from paper_2506_12038_amd.binding import GemvGroup
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256
    layer = synth.make_layer_uniform(N, K, bits, M, seed=N + K + M)
    packed, lut = lcd.lcd_pack_indices(to_dev(layer["idx"]), bits), lcd.lcd_build_lut(to_dev(layer["codebook"]), bits)
    x, s = to_dev(layer["x"]), to_dev(layer["s"])
    x2, half = (x * 0.5).contiguous(), (M + 1) // 2      # (halves: a part of one or two tokens could be the bucket kernel's)

    def parts(a):
        ys = []
        for m in range(0, M, half):
            ws = _WatchedWorkspace(lcd.lcd_workspace_bytes(half, N, K, bits))
            ys.append(lcd.lcd_lut_gemv(packed, lut, a[m:m + half].contiguous(), s, N, bits, workspace=ws.tensor))
            assert not ws.written()
        return torch.cat(ys)

    ref, ref2 = parts(x), parts(x2)
    ws = _WatchedWorkspace(lcd.lcd_workspace_bytes(M, N, K, bits))
    y = lcd.lcd_lut_gemv(packed, lut, x, s, N, bits, workspace=ws.tensor)
    assert ws.written() == ahead[0]
    assert torch.equal(y, ref)
    outs = [torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2)]
    problems = [(packed, lut, x, s, outs[0], N), (packed, lut, x2, s, outs[1], N)]
    ws = _WatchedWorkspace(GemvGroup(problems, bits).workspace.numel())
    GemvGroup(problems, bits, workspace=ws.tensor)()
    assert ws.written() == ahead[1]
    assert torch.equal(outs[0], ref) and torch.equal(outs[1], ref2)
    rows = np.unique(np.linspace(0, N - 1, 48).astype(int))
    assert_parity(y.cpu().numpy()[:, rows], oracle.lut_matmul(layer["codebook"][rows], layer["idx"][rows], layer["x"], layer["s"], bits), TOL)
