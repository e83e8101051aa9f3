"""GPU: the decode entry points on layers of 2^27 columns and more (one row tile: 16 rows), where 32-bit sums and offsets end."""
import numpy as np
import pytest

import synth
import paper_2506_12038_amd as lcd
from gpu_common import TOL, assert_parity, to_dev

pytestmark = pytest.mark.gpu

Q8_TOL = 1e-3   # codes are exact matrix operands: only the fp32 accumulation and the fp16 store differ from the fp64 sum
ROWS, WIDE = 16, 1 << 27


@pytest.fixture(autouse=True)
def _give_memory_back():
    import torch
    yield
    torch.cuda.empty_cache()


def _workspace(M, K, bits):
    import torch
    return torch.empty(lcd.lcd_workspace_bytes(M, ROWS, K, bits), dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("bits,M", [(2, 1), (2, 4), (3, 1)])
@pytest.mark.parametrize("K", [WIDE, WIDE + 2048])
def test_q8_sums_of_the_largest_codes_in_one_bucket(bits, M, K):
    # every code at a limit of its range, every weight in one cluster: a bucket's sum is -2^31 per eighth of 2^27 columns.
    # Single calls of both entry points, and grouped with a layer of ordinary size, whose bits must not depend on its neighbour.
    import torch
    from paper_2506_12038_amd.binding import GemvGroup
    s_q, centroid = 2.0 ** -10, 2.0 ** -14
    codes = np.array([-128, 127, -128, 127][:M])
    x = torch.from_numpy((codes * s_q).astype(np.float16)).cuda()[:, None].expand(M, K).contiguous()
    s = torch.ones(K, dtype=torch.float32, device="cuda")
    packed = lcd.lcd_pack_indices(torch.ones((ROWS, K), dtype=torch.uint8, device="cuda"), bits)
    codebook = torch.zeros((ROWS, 1 << bits), dtype=torch.float16, device="cuda")
    codebook[:, 1] = centroid
    lut = lcd.lcd_build_lut(codebook, bits)
    Y = np.repeat((s_q * centroid * K * codes)[:, None], ROWS, axis=1)
    ws = _workspace(M, K, bits)
    for entry in (lcd.lcd_lut_gemv_q8, lcd.lcd_lut_gemm_q8):
        assert_parity(entry(packed, lut, x, s, s_q, ROWS, bits, workspace=ws).cpu().numpy(), Y, Q8_TOL, entry.__name__)
    del ws
    layer = synth.make_layer(1, 0, 48, 1280, bits, M)
    usual = (lcd.lcd_pack_indices(to_dev(layer["idx"]), bits), lcd.lcd_build_lut(to_dev(layer["codebook"]), bits), to_dev(layer["x"]), to_dev(layer["s"]))
    outs = [torch.full((M, n), float("nan"), dtype=torch.float16, device="cuda") for n in (48, ROWS)]
    GemvGroup([(*usual, outs[0], 48), (packed, lut, x, s, outs[1], ROWS)], bits, s_q=[0.05, s_q])()
    assert torch.equal(outs[0], lcd.lcd_lut_gemv_q8(*usual, 0.05, 48, bits))
    assert_parity(outs[1].cpu().numpy(), Y, Q8_TOL)


@pytest.mark.parametrize("bits,M", [(2, 1), (2, 2), (3, 1)])
@pytest.mark.parametrize("K", [1 << 21, (1 << 21) + 4096, WIDE + 2048])
def test_bucket_sums_of_equal_activations(bits, M, K):
    # every addition of a run has the same sign and loses a part of the same sign (a quarter of 32.25 beyond 2^22): 2^12 of them lose 2^-12 at most
    import torch
    value, centroid = 1.0078125, 2.0 ** -14 if K > WIDE else 2.0 ** -8
    x = torch.full((M, K), value, dtype=torch.float16, device="cuda")
    x[M - 1] *= -1
    s = torch.ones(K, dtype=torch.float32, device="cuda")
    packed = lcd.lcd_pack_indices(torch.ones((ROWS, K), dtype=torch.uint8, device="cuda"), bits)
    codebook = torch.zeros((ROWS, 1 << bits), dtype=torch.float16, device="cuda")
    codebook[:, 1] = centroid
    y = lcd.lcd_lut_gemv(packed, lcd.lcd_build_lut(codebook, bits), x, s, ROWS, bits, workspace=_workspace(M, K, bits))
    assert_parity(y.cpu().numpy(), x[:, :1].double().cpu().numpy() * K * np.full((1, ROWS), centroid), TOL)


@pytest.mark.parametrize("bits,M,quantised", [(2, 16, False), (2, 16, True), (3, 15, False), (4, 16, False)])
def test_activations_of_four_gibibytes(bits, M, quantised):
    # 16 tokens of 2^27 columns are 2^32 bytes, one more than the kernels' 32-bit offsets reach (15 tokens fit).  All but some columns
    # are zero, the first and the last of every token are not.  Single call, and grouped with a layer of ordinary size.
    import torch
    from paper_2506_12038_amd.binding import GemvGroup
    K, g = WIDE, torch.Generator(device="cuda")
    g.manual_seed(17 * bits + M)
    idx = torch.randint(0, 1 << bits, (ROWS, K), dtype=torch.uint8, device="cuda", generator=g)
    columns = torch.randint(0, K, (M, 512), device="cuda", generator=g)
    columns[:, 0], columns[:, 1] = 0, K - 1
    s_q = 2.0 ** -5
    values = torch.randint(-100, 100, (M, 512), device="cuda", generator=g).half() * s_q        # (the codes themselves, s = 1)
    x = torch.zeros((M, K), dtype=torch.float16, device="cuda").scatter_(1, columns, values)
    s = torch.ones(K, dtype=torch.float32, device="cuda")
    codebook = (torch.randn((ROWS, 1 << bits), device="cuda", generator=g) * 0.02).half()
    weights = torch.stack([codebook.double().gather(1, idx[:, c].long()) for c in columns])      # [M, rows, 512]
    Y = (weights * x.gather(1, columns).double()[:, None, :])
    # (a column drawn twice counts once)
    first = torch.stack([torch.isin(torch.arange(512, device="cuda"), torch.from_numpy(np.unique(c.cpu().numpy(), return_index=True)[1]).cuda()) for c in columns])
    Y = (Y * first[:, None, :]).sum(dim=2).cpu().numpy()
    packed, lut = lcd.lcd_pack_indices(idx, bits), lcd.lcd_build_lut(codebook, bits)
    del idx, weights
    ws = _workspace(M, K, bits)
    call = (lambda a, n: lcd.lcd_lut_gemv_q8(*a, s_q, n, bits, workspace=ws)) if quantised else (lambda a, n: lcd.lcd_lut_gemv(*a, n, bits, workspace=ws))
    y = call((packed, lut, x, s), ROWS)
    assert_parity(y.cpu().numpy(), Y, TOL)
    layer = synth.make_layer(1, 0, 48, 1280, bits, M)
    usual = (lcd.lcd_pack_indices(to_dev(layer["idx"]), bits), lcd.lcd_build_lut(to_dev(layer["codebook"]), bits), to_dev(layer["x"]), to_dev(layer["s"]))
    outs = [torch.full((M, n), float("nan"), dtype=torch.float16, device="cuda") for n in (48, ROWS)]
    problems = [(*usual, outs[0], 48), (packed, lut, x, s, outs[1], ROWS)]
    GemvGroup(problems, bits, s_q=[s_q, s_q] if quantised else None)()
    assert torch.equal(outs[0], call(usual, 48)) and torch.equal(outs[1], y)
