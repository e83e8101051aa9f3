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
