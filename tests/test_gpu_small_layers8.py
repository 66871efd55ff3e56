"""The small-layer kernel on 8-bit activations: each shape of it, int8 (exact sums: outputs equal the
oracle's bit for bit) and fp8 (within the bound derived from the matrix core's window), on layers at the
edges of its tiles: one row, 31 to 33 rows, filter counts around 32 and 64 and no multiple of 4, fewer
stages than waves and many more, odd numbers of 64-element code chunks, taps on every border, strides.
"""
import numpy as np
import pytest

import oracle
import test_gpu_fp8 as fp8
import test_gpu_i8 as i8
from test_gpu_parity import log

pytestmark = pytest.mark.gpu

# n, h, w, c, k, r, s, stride, pad
CASES = [(1, 1, 1, 16, 1, 1, 1, 1, 0), (1, 1, 31, 16, 32, 1, 1, 1, 0), (1, 1, 33, 128, 33, 1, 1, 1, 0),
         (2, 5, 7, 48, 66, 3, 3, 1, 1), (1, 7, 7, 128, 100, 3, 3, 2, 1), (3, 4, 4, 80, 31, 5, 5, 1, 2),
         (2, 6, 5, 192, 65, 3, 1, 1, 2), (1, 9, 9, 16, 96, 7, 7, 1, 3), (1, 3, 3, 1024, 40, 3, 3, 1, 1)]


@pytest.mark.parametrize("tile", [-1, 5, 6, 7, 8])
def test_small_layers_8bit(tbn, tile, knobs):
    knobs(i8_tile=tile, fp8_tile=tile)
    for g in CASES:
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
