"""The kernel for 3 x 3 layers of stride 1 over 64 channels, on layers at the edges of its units (4 x 8
output pixels) and filter groups (32): one pixel, maps one more and one less than whole units, taps
on every border, pads of 0 to 2, filter counts that fill a group partly, ranges of units that cross
images, more waves than units -- against the fp64 oracle, forward with and without the whole epilogue
and backward-data 1e-2 (normalised max error, bf16 outputs), and against the tiled kernel, whose sums it
forms in the same order (bf16 outputs at most one unit in the last place apart: 2^-7 of the value).
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from test_gpu_parity import TOL, bf16_dev, log, nerr, to_dev

pytestmark = pytest.mark.gpu

# n, h, w, k, pad; the backward pass has 64 filters and k channels
CASES = [(1, 1, 1, 8, 1), (1, 4, 8, 32, 1), (2, 5, 9, 40, 1), (3, 3, 7, 64, 1), (1, 12, 17, 72, 0), (2, 9, 6, 24, 2),
         (5, 13, 11, 200, 1)]
# ... and on either side of the rule that chooses it
RULE = [(9, 28, 28, 64, 1), (30, 28, 28, 64, 1), (21, 41, 38, 64, 1), (12, 56, 56, 64, 1), (40, 30, 31, 104, 1),
        (48, 26, 26, 64, 1), (50, 26, 26, 64, 1), (29, 33, 33, 40, 1), (159, 26, 25, 64, 1), (126, 27, 27, 64, 1),
        (87, 29, 29, 128, 1), (136, 26, 26, 128, 1)]


def _check(tbn, case, knobs, forced):
    n, h, w, k, pad = case
    log("64-channel layer %s %s" % (case, forced))
    g = (n, h, w, 64, k, 3, 3, 1, pad)
    d, desc = oracle.ConvDesc(*g), tbn.ConvDesc(*g)
    P, Q = d.out_dims()
    xb = synth.normal_bf16(9, "cx%s" % (g,), (n, h, w, 64))
    wr = synth.normal(9, "cw%s" % (g,), (k, 576), 1.0)
    resb = synth.normal_bf16(9, "cr%s" % (g,), (n, P, Q, k))
    scale, bias = synth.uniform(9, "cs%s" % (g,), (k,), 0.5, 1.5), synth.normal(9, "cb%s" % (g,), (k,), 0.1)
    codes, alpha, _ = tbn.quantize(to_dev(wr))
    x, res = bf16_dev(xb), bf16_dev(resb)
    # backward: 64 filters, so that the gradient has 64 channels, over k input channels
    gb = (n, h, w, k, 64, 3, 3, 1, pad)
    db, descb = oracle.ConvDesc(*gb), tbn.ConvDesc(*gb)
    dyb = synth.normal_bf16(9, "cdy%s" % (g,), (n, P, Q, 64))
    wb = synth.normal(9, "cwb%s" % (g,), (64, 9 * k), 1.0)
    codes_b, alpha_b, _ = tbn.quantize(to_dev(wb))
    dy = bf16_dev(dyb)

    def run():
        out = [tbn.conv2d_fwd(desc, x, codes, alpha),
               tbn.conv2d_fwd(desc, x, codes, alpha, scale=to_dev(scale), bias=to_dev(bias), residual=res, relu=True),
               tbn.conv2d_bwd_data(descb, dy, codes_b, alpha_b)]
        torch.cuda.synchronize()
        return [o.float().cpu().numpy() for o in out]

    knobs(conv_tile=forced)
    got = run()
    knobs(conv_tile=14)
    tiled = run()
    for a, b in zip(got, tiled):
        assert np.all(np.abs(a - b) <= np.maximum(np.abs(a), np.abs(b)) * 2.0 ** -7 + 1e-6 * np.abs(b).max())
    if n * P * Q * k <= 40000:
        q, qb = oracle.quantize(wr), oracle.quantize(wb)
        acc = oracle.conv_fwd(d, oracle.bf16_bits_to_f64(xb), q.codes, q.alpha.astype(np.float64))
        full = np.maximum(acc * scale.astype(np.float64) + bias + oracle.bf16_bits_to_f64(resb), 0.0)
        dx = oracle.conv_bwd_data(db, oracle.bf16_bits_to_f64(dyb), qb.codes, qb.alpha.astype(np.float64))
        for a, ref in zip(got, (acc, full, dx)):
            assert nerr(a, ref) <= TOL


@pytest.mark.parametrize("case", CASES)
def test_c64_edges(tbn, case, knobs):
    _check(tbn, case, knobs, 60)


@pytest.mark.parametrize("case", RULE)
def test_c64_rule(tbn, case, knobs):
    _check(tbn, case, knobs, -1)
