"""The small-layer kernel on 8-bit activations: each shape of it, int8 (exact sums: outputs equal the
oracle's bit for bit) and fp8 (within the bound derived from the matrix core's window), on layers at the
edges of its tiles: one row, 31 to 33 rows, filter counts around 32 and 64 and no multiple of 4, fewer
stages than waves and many more, odd numbers of 64-element code chunks, taps on every border, strides.
And the E4M3 codes of fp32 values over all exponents, the halfway cases among them.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
import test_gpu_fp8 as fp8
import test_gpu_i8 as i8
from test_gpu_parity import log, to_dev

pytestmark = pytest.mark.gpu

# n, h, w, c, k, r, s, stride, pad
CASES = [(1, 1, 1, 16, 1, 1, 1, 1, 0), (1, 1, 31, 16, 32, 1, 1, 1, 0), (1, 1, 33, 128, 33, 1, 1, 1, 0),
         (2, 5, 7, 48, 66, 3, 3, 1, 1), (1, 7, 7, 128, 100, 3, 3, 2, 1), (3, 4, 4, 80, 31, 5, 5, 1, 2),
         (2, 6, 5, 192, 65, 3, 1, 1, 2), (1, 9, 9, 16, 96, 7, 7, 1, 3), (1, 3, 3, 1024, 40, 3, 3, 1, 1)]

# ... and where the built-in choice changes beyond them: 64 and 65 filters with fewer than 384 tiles, and with more;
# 33 and 64 filters with 256 tiles of 64 rows and with 257
RULE = [(1, 131, 129, 16, 64, 1, 1, 1, 0), (1, 131, 129, 16, 65, 1, 1, 1, 0), (1, 131, 129, 16, 31, 3, 3, 1, 1),
        (1, 222, 223, 16, 64, 1, 1, 1, 0), (1, 222, 223, 16, 65, 1, 1, 1, 0), (1, 128, 128, 16, 64, 3, 3, 1, 1), (1, 113, 145, 16, 64, 3, 3, 1, 1),
        (1, 128, 128, 16, 33, 1, 1, 1, 0), (1, 113, 145, 32, 33, 1, 1, 1, 0)]


@pytest.mark.parametrize("tile", [-1, 5, 6, 7])
def test_small_layers_8bit(tbn, tile, knobs):
    knobs(i8_tile=tile, fp8_tile=tile)
    for g in CASES + (RULE if tile < 0 else []):
        for out, relu in (("f32", False), ("bf16", True)):
            log("small 8-bit layer %s shape %d %s" % (g, tile, out))
            d, xq, codes, alpha, words, x_scale = i8._problem(g, 4)
            ref, _ = oracle.conv_fwd_i8(d, xq, codes, alpha, x_scale, relu=relu)
            got = i8._run(tbn, g, xq, words, alpha, x_scale, out, relu)
            assert np.array_equal(got.astype(np.float64), i8._expect(ref, out).reshape(got.shape))
            d, xq, codes, alpha, words, x_scale = fp8._problem(g, 4)
            ref = oracle.conv_fwd_fp8(d, xq, codes, alpha, x_scale, relu=relu)
            got = fp8._run(tbn, g, xq, words, alpha, x_scale, out, relu)
            fp8.check(got, ref.reshape(got.shape), d, xq, alpha, x_scale, out)


def test_fp8_codes_of_fp32_values(tbn):
    g = synth.rng(9, "fp8 fp32 values")
    bits = g.integers(0, 1 << 32, size=1 << 18, dtype=np.uint64).astype(np.uint32)  # every exponent, NaN, inf
    near = (g.integers(0, 1 << 24, size=1 << 18) / np.float64(1 << 15)).astype(np.float32)  # 0 .. 512 in 2^-15
    half = np.concatenate([np.arange(0, 1 << 12) * np.float32(2.0 ** -11), np.arange(0, 1 << 10) * np.float32(0.5)])
    x = np.concatenate([bits.view(np.float32), near, -near, half.astype(np.float32), -half.astype(np.float32)])
    for inv in (np.float32(1.0), np.float32(0.37)):
        log("fp8 codes of %d fp32 values, inverse scale %g" % (x.size, inv))
        got = tbn.quantize_act_fp8(to_dev(x), float(inv))
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), oracle.quantize_act_fp8(x, inv))
