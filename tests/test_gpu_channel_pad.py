"""Layers whose channel counts are no multiple of 8, which run on zero-padded copies of their
tensors: every remainder of C and K against 8, runs of codes that cross packed words, odd element
offsets and an odd element count (the last word of a tensor read as 2 bytes), 1 x 1 and strided
windows, against the fp64 oracle at the bars of the parity suite (forward with fp32 output and filter
gradient 1e-4, gradient to the input 1e-2, normalised max error).  The same calls with only the
workspace that the unpadded layer needs take the general kernels and agree.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from test_gpu_parity import bf16_dev, log, nerr, to_dev

pytestmark = pytest.mark.gpu

# n, h, w, c, k, r, s, stride, pad
CASES = [(1, 1, 1, 9, 3, 1, 1, 1, 0), (2, 5, 7, 9, 9, 3, 3, 1, 1), (1, 3, 3, 10, 15, 1, 1, 1, 0),
         (3, 6, 5, 11, 66, 3, 3, 1, 1), (2, 9, 4, 12, 20, 5, 5, 1, 2), (1, 7, 7, 13, 64, 3, 3, 1, 1),
         (2, 6, 6, 23, 7, 3, 3, 2, 1), (1, 5, 9, 36, 100, 3, 3, 1, 1), (2, 4, 4, 63, 8, 3, 1, 1, 0),
         (1, 4, 5, 65, 129, 3, 3, 1, 1), (2, 8, 8, 5, 10, 3, 3, 1, 1), (1, 1, 1, 1001, 33, 1, 1, 1, 0)]


def _legacy(g):
    """Bytes of the unpadded layer's backward-data workspace: re-packed codes and scale pairs."""
    n, h, w, c, k, r, s, _, _ = g
    blocks = (r * s * k + 63) // 64
    return ((c + 63) // 64 * blocks * 1024 + 255) // 256 * 256 + (blocks * 128 + 255) // 256 * 256


@pytest.mark.parametrize("g", CASES, ids=str)
def test_ragged_channels(tbn, g):
    log("ragged channels %s" % (g,))
    n, h, w, c, k, r, s, stride, _ = g
    d, desc = oracle.ConvDesc(*g), tbn.ConvDesc(*g)
    P, Q = d.out_dims()
    xb = synth.normal_bf16(9, "px%s" % (g,), (n, h, w, c))
    dyb = synth.normal_bf16(9, "pdy%s" % (g,), (n, P, Q, k))
    wr = synth.normal(9, "pw%s" % (g,), (k, r * s * c), 1.0)
    q = oracle.quantize(wr)
    alpha64 = q.alpha.astype(np.float64)
    x64, dy64 = oracle.bf16_bits_to_f64(xb), oracle.bf16_bits_to_f64(dyb)
    codes, alpha, _ = tbn.quantize(to_dev(wr))
    x, dy = bf16_dev(xb), bf16_dev(dyb)
    small = torch.empty(16, dtype=torch.uint8, device="cuda")

    ref = oracle.conv_fwd(d, x64, q.codes, alpha64)
    for xin in (x, x.float()):
        for ws in (None, small) if c > 8 else (None,):
            y = tbn.conv2d_fwd(desc, xin, codes, alpha, out_dtype=torch.float32, ws=ws)
            torch.cuda.synchronize()
            assert nerr(y.cpu().numpy(), ref) <= 1e-4

    ref = oracle.conv_bwd_weight(d, x64, dy64)
    dw = tbn.conv2d_bwd_weight(desc, x, dy)
    twice = tbn.conv2d_bwd_weight(desc, x, dy, dw=dw.clone(), accumulate=True)
    torch.cuda.synchronize()
    assert nerr(dw.cpu().numpy(), ref) <= 1e-4
    assert nerr(twice.cpu().numpy(), 2 * ref) <= 1e-4

    if stride == 1:
        ref = oracle.conv_bwd_data(d, dy64, q.codes, alpha64)
        for ws in (None,) + ((torch.empty(_legacy(g), dtype=torch.uint8, device="cuda"),) if c % 8 and k % 8 else ()):
            dx = tbn.conv2d_bwd_data(desc, dy, codes, alpha, out_dtype=torch.float32, ws=ws)
            torch.cuda.synchronize()
            assert nerr(dx.cpu().numpy(), ref) <= 1e-2
