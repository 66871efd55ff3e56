"""The small-layer convolution kernel: every shape of it on layers at the edges of its tiles (one
row, 31 to 33 rows, filter counts on either side of 32 and 64 and no multiple of 4, fewer stages than
waves, many more, a last stage that is partial, taps on every border, strides) against the fp64 oracle:
forward with fp32 output 1e-4, with the whole bf16 epilogue and backward-data 1e-2 (normalised max
error); and the layers on either side of the rule that chooses it.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from test_gpu_parity import TOL, bf16_dev, log, nerr, to_dev

pytestmark = pytest.mark.gpu

# n, h, w, c, k, r, s, stride, pad
CASES = [(1, 1, 1, 8, 1, 1, 1, 1, 0), (1, 1, 31, 16, 32, 1, 1, 1, 0), (1, 1, 32, 64, 33, 1, 1, 1, 0),
         (1, 3, 11, 64, 64, 3, 3, 1, 1), (2, 5, 7, 24, 66, 3, 3, 1, 1), (1, 7, 7, 128, 100, 3, 3, 2, 1),
         (3, 4, 4, 40, 31, 5, 5, 1, 2), (2, 6, 5, 192, 65, 3, 1, 1, 2), (1, 9, 9, 8, 96, 7, 7, 1, 3),
         (33, 1, 1, 1160, 10, 1, 1, 1, 0), (1, 2, 2, 512, 40, 2, 2, 1, 0)]
# ... where the built-in rule changes between the shapes and the tiled kernel
RULE = [(1, 8, 32, 64, 1024, 1, 1, 1, 0), (1, 8, 33, 64, 1024, 1, 1, 1, 0), (1, 8, 33, 512, 1024, 3, 1, 1, 0),
        (17, 1, 1, 12800, 12, 1, 1, 1, 0), (17, 1, 1, 12808, 12, 1, 1, 1, 0), (5, 21, 19, 96, 320, 3, 3, 1, 1)]


def _check(tbn, g, what):
    log("small layer %s %s" % (g, what))
    n, h, w, c, k, r, s, stride, _ = g
    d, desc = oracle.ConvDesc(*g), tbn.ConvDesc(*g)
    P, Q = d.out_dims()
    xb = synth.normal_bf16(9, "sx%s" % (g,), (n, h, w, c))
    dyb = synth.normal_bf16(9, "sdy%s" % (g,), (n, P, Q, k))
    wr = synth.normal(9, "sw%s" % (g,), (k, r * s * c), 1.0)
    resb = synth.normal_bf16(9, "sr%s" % (g,), (n, P, Q, k))
    scale, bias = synth.uniform(9, "ss%s" % (g,), (k,), 0.5, 1.5), synth.normal(9, "sb%s" % (g,), (k,), 0.1)
    q = oracle.quantize(wr)
    a64 = q.alpha.astype(np.float64)
    acc = oracle.conv_fwd(d, oracle.bf16_bits_to_f64(xb), q.codes, a64)
    full = np.maximum(acc * scale.astype(np.float64) + bias + oracle.bf16_bits_to_f64(resb), 0.0)
    codes, alpha, _ = tbn.quantize(to_dev(wr))
    x = bf16_dev(xb)
    kw = dict(scale=to_dev(scale), bias=to_dev(bias), relu=True)
    y32 = tbn.conv2d_fwd(desc, x, codes, alpha, out_dtype=torch.float32)
    y = tbn.conv2d_fwd(desc, x, codes, alpha, residual=bf16_dev(resb), **kw)
    f32 = tbn.conv2d_fwd(desc, x, codes, alpha, residual=bf16_dev(resb).float(), out_dtype=torch.float32, **kw)
    torch.cuda.synchronize()
    assert nerr(y32.cpu().numpy(), acc) <= 1e-4
    assert nerr(y.float().cpu().numpy(), full) <= TOL
    assert nerr(f32.cpu().numpy(), full) <= 1e-4
    if stride == 1:
        dx = tbn.conv2d_bwd_data(desc, bf16_dev(dyb), codes, alpha, out_dtype=torch.float32)
        torch.cuda.synchronize()
        assert nerr(dx.cpu().numpy(), oracle.conv_bwd_data(d, oracle.bf16_bits_to_f64(dyb), q.codes, a64)) <= TOL


@pytest.mark.parametrize("tile", [51, 52, 53, 54, 55])
def test_small_layer_shapes(tbn, tile, knobs):
    knobs(conv_tile=tile)
    for g in CASES:
        _check(tbn, g, "shape %d" % tile)


def test_small_layer_rule(tbn):
    for g in CASES + RULE:
        _check(tbn, g, "built-in choice")


def test_one_row_backward_beyond_the_small_layers(tbn):
    # a window as large as its input and 201 stages: backward-data of it is split over the grid
    for g in [(1, 1, 1, 72, 12808, 1, 1, 1, 0), (1, 1, 1, 256, 16384, 1, 1, 1, 0), (1, 1, 1, 40, 3216, 2, 2, 1, 1)]:
        _check(tbn, g, "one row")
