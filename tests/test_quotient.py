"""The quantiser's quotient (csrc/lcd_device.h: refined reciprocal, product, one residual correction) at the places where a code could change.

A code can only differ from the correctly rounded quotient's where x / (s * s_q) lies within rounding of a half-integer.  CPU: every fp16
significand, every half-integer up to 128.5, the divisors within 8 ulps of their quotient, hardware reciprocals off by one ulp either way, one
correction against two and against the binary32 division.  GPU: such places through every kernel that quantises, against the oracle.
"""
import shutil
import subprocess

import numpy as np
import pytest

import oracle
import paper_2506_12038_amd as lcd
from gpu_common import to_dev

SWEEP = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
static float step(float f, int ulps) { uint32_t u; memcpy(&u, &f, 4); u += (uint32_t)ulps; memcpy(&f, &u, 4); return f; }
static float quotient(float x, float d, float y0, int corrections)
{
    const float y = std::fma(std::fma(-d, y0, 1.0f), y0, y0);
    float q = x * y;
    for (int i = 0; i < corrections; ++i) q = std::fma(std::fma(-d, q, x), y, q);
    return q;
}
static int code(float q) { return (int)std::nearbyint(std::fmin(std::fmax(q, -128.0f), 127.0f)); }
int main()
{
    long places = 0, one_from_two = 0, wrong = 0, wrong_exact_reciprocal = 0, wrong_elsewhere = 0;
    for (int m = 1024; m < 2048; ++m)
        for (int h = 0; h <= 128; ++h) {
            const float x = (float)m, near_d = (float)((double)x / (h + 0.5));
            for (int k = -8; k <= 8; ++k) {
                const float d = step(near_d, k), r = (float)(1.0 / (double)d);
                int e;
                const bool ones = std::frexp(d, &e) == 1.0f - std::ldexp(1.0f, -24);     // the largest significand
                for (int off = -1; off <= 1; ++off) {
                    const int one = code(quotient(x, d, step(r, off), 1)), two = code(quotient(x, d, step(r, off), 2)), ieee = code(x / d);
                    ++places;
                    one_from_two += one != two;
                    wrong += one != ieee;
                    wrong_exact_reciprocal += one != ieee && off == 0;
                    wrong_elsewhere += one != ieee && !(ones && m == 1024 && h == 0);
                }
            }
        }
    std::printf("%ld %ld %ld %ld %ld\n", places, one_from_two, wrong, wrong_exact_reciprocal, wrong_elsewhere);
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_one_correction_decides_every_code_like_two_and_like_the_division(tmp_path):
    (tmp_path / "sweep.cpp").write_text(SWEEP)
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-ffp-contract=off", str(tmp_path / "sweep.cpp"), "-o", str(tmp_path / "sweep")])
    out = subprocess.run([str(tmp_path / "sweep")], capture_output=True, text=True, timeout=120, check=True).stdout
    places, one_from_two, wrong, wrong_exact_reciprocal, wrong_elsewhere = map(int, out.split())
    assert places == 1024 * 129 * 17 * 3
    assert one_from_two == 0
    # one place needs the reciprocal correctly rounded: a divisor of the largest significand under a power of two, just above one half
    assert wrong_exact_reciprocal == 0 and wrong_elsewhere == 0 and wrong == 2


def _hard_columns(K, seed):
    """K columns: an fp16 number and a divisor whose quotient lies within a few ulps of a half-integer, the powers of two over the largest
    significand among them."""
    rng = np.random.default_rng(seed)
    half = rng.integers(0, 129, K)
    x = rng.integers(1024, 2048, K).astype(np.float64)
    d = (x / (half + 0.5)).astype(np.float32)
    d = (d.view(np.uint32) + rng.integers(-3, 4, K).astype(np.int64)).astype(np.uint32).view(np.float32)
    x[:64], d[:64] = 1024.0, np.nextafter(np.float32(2048.0), np.float32(0.0))
    scale = 2.0 ** rng.integers(-12, 5, K)
    return (x * scale * rng.choice([-1.0, 1.0], K)).astype(np.float16), (d * scale.astype(np.float32)).astype(np.float32)


@pytest.mark.gpu
@pytest.mark.parametrize("M", [1, 2, 3, 4, 7, 16, 40, 200, 2100])
def test_gpu_codes_next_to_half_integers(M):
    # row n reads column n: y = s_q * q, s_q a power of two.  1 to 4 tokens: the bucket kernel's codes; 7: the tokens kernel's (16 at K = 4096: made
    # ahead); 40: ahead of the narrow kernel; 200 and 2100: ahead of the split and the wide tiles.
    import torch
    bits, K = 2, 4096
    codebook = np.zeros((K, 4), dtype=np.float16)
    codebook[:, 0] = 1.0
    idx = np.ones((K, K), dtype=np.uint8)
    idx[np.arange(K), np.arange(K)] = 0
    packed, lut = lcd.lcd_pack_indices(to_dev(idx), bits), lcd.lcd_build_lut(to_dev(codebook), bits)
    entry = lcd.lcd_lut_gemv_q8 if M <= 16 else lcd.lcd_lut_gemm_q8
    for seed in range(4):
        row, d = _hard_columns(K, seed)
        s_q = 0.125
        x, s = np.repeat(row[None, :], M, axis=0), d * np.float32(8.0)
        x[1::2] *= -1
        q = oracle.input_transform(x[:2], s, s_q, 8, single_precision=True)
        y = entry(packed, lut, to_dev(x), to_dev(s), s_q, K, bits)
        torch.cuda.synchronize()
        got = y.cpu().numpy().astype(np.float64) / s_q
        for m in range(M):
            assert np.array_equal(got[m], q[m % 2].astype(np.float64)), (seed, m, np.flatnonzero(got[m] != q[m % 2])[:8])
