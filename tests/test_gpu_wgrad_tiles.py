"""The narrow-tile filter-gradient kernel at the edges of its tiles: K and J on either side of each tile
(32, 64, 128 and 256 filters; 64 and 256 columns), pixel counts that end inside a stage, in the first
group's half and with the second group empty, strides, uneven windows, one pixel; against the fp64
oracle (fp32 sums of exact bf16 products: 1e-4 normalised max error, as in the parity suite), the same
bits on a second call, and added to a prior gradient.  Every case also runs on the 256 x 256 kernel; and
the built-in choice where it takes tiles of fewer filters than a layer has.
"""
import pytest
import torch

import oracle
import synth
from test_gpu_parity import bf16_dev, log, nerr

pytestmark = pytest.mark.gpu

# n, h, w, c, k, r, s, stride, pad
CASES = [(1, 1, 1, 8, 8, 1, 1, 1, 0), (1, 3, 11, 64, 64, 1, 1, 1, 0), (2, 8, 8, 72, 64, 1, 1, 1, 0),
         (1, 5, 13, 8, 72, 1, 1, 1, 0), (1, 16, 16, 8, 264, 3, 2, 1, 1), (3, 7, 5, 32, 32, 3, 3, 1, 1),
         (2, 9, 9, 32, 40, 3, 3, 2, 1), (1, 33, 31, 40, 128, 3, 3, 1, 1), (5, 6, 7, 104, 24, 1, 3, 2, 0),
         (2, 4, 4, 256, 8, 4, 4, 1, 0), (4, 14, 14, 32, 64, 5, 5, 1, 2), (1, 2, 200, 16, 96, 2, 1, 1, 1)]

# 97 column tiles (3 x 3 over 2736 channels), one chunk of pixels: tiles of 32, 64 and 256 filters for 40, 128 and 512;
# 53 column tiles and seven chunks: 128 for 384; just over 64 columns, and up to 64, with few and with many filters
RULE = [(1, 8, 8, 2736, 40, 3, 3, 1, 1), (1, 8, 8, 2736, 128, 3, 3, 1, 1), (1, 8, 8, 2736, 512, 3, 3, 1, 1),
        (1, 21, 21, 536, 384, 5, 5, 1, 2), (2, 5, 5, 8, 104, 3, 3, 1, 1), (24, 24, 24, 8, 296, 3, 3, 1, 1),
        (2, 9, 7, 24, 264, 1, 1, 1, 0)]


@pytest.mark.parametrize("g", CASES, ids=str)
def test_wgrad_narrow_tiles(tbn, g, knobs):
    _check(tbn, g, knobs, (-1, 0, 1))


@pytest.mark.parametrize("g", RULE, ids=str)
def test_wgrad_tile_rule(tbn, g, knobs):
    _check(tbn, g, knobs, (-1,))


def _check(tbn, g, knobs, kernels):
    n, h, w, c, k = g[:5]
    d, desc = oracle.ConvDesc(*g), tbn.ConvDesc(*g)
    P, Q = d.out_dims()
    xb = synth.normal_bf16(9, "nx%s" % (g,), (n, h, w, c))
    dyb = synth.normal_bf16(9, "ndy%s" % (g,), (n, P, Q, k))
    ref = oracle.conv_bwd_weight(d, oracle.bf16_bits_to_f64(xb), oracle.bf16_bits_to_f64(dyb))
    x, dy = bf16_dev(xb), bf16_dev(dyb)
    for cfg in kernels:
        log("narrow filter gradient %s, kernel %d" % (g, cfg))
        knobs(wgrad_cfg=cfg)
        dw = tbn.conv2d_bwd_weight(desc, x, dy)
        again = tbn.conv2d_bwd_weight(desc, x, dy)
        twice = tbn.conv2d_bwd_weight(desc, x, dy, dw=dw.clone(), accumulate=True)
        torch.cuda.synchronize()
        assert nerr(dw.cpu().numpy(), ref) <= 1e-4
        assert torch.equal(dw, again)
        assert nerr(twice.cpu().numpy(), 2 * ref) <= 1e-4


def test_wgrad_window_of_more_than_32768_rows(tbn):
    # 28 of the 32 rows of the only stage are no pixels: at tap 32768 they must not reach back into the
    # images (x element 32768 * 8 on, infinite here), whatever dy they are multiplied with (zeros)
    log("filter gradient, window of 33000 rows")
    n, h, r, pad = 4, 10000, 33000, 11500
    desc = tbn.ConvDesc(n, h, 1, 8, 8, r, 1, 1, pad, pad_w=0)
    assert desc.out_dims() == (1, 1)
    g = torch.Generator().manual_seed(3)
    x, dy = torch.randn(n, h, 8, generator=g).bfloat16(), torch.randn(n, 8, generator=g).bfloat16()
    flat = x.view(-1, 8)
    flat[32768] = float("inf")  # row 2768 of image 3: tap 14268 sees it
    want = torch.zeros(8, r, 8, dtype=torch.float64)
    want[:, pad:pad + h] = torch.einsum("nk,nhc->khc", dy.double(), x.double())
    got = tbn.conv2d_bwd_weight(desc, x.cuda(), dy.cuda()).cpu().double().view(8, r, 8)
    hit = ~torch.isfinite(want)
    assert torch.equal(~torch.isfinite(got), hit)
    assert float((got - want)[~hit].abs().max()) <= 1e-4 * float(want[~hit].abs().max())
