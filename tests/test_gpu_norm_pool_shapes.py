"""Batch normalisation at row and channel counts around its thread layouts (8 channels per thread, 8
values over uneven channel counts with every remainder of rows against 8, one channel per thread; one
row, chunks with remainders of the unrolled steps, several slices of channels), and pooling backward over
windows that do not overlap, with input rows and columns past the last window, on both sides of the size from
which windows and not inputs are walked.  Against fp64 torch:
the layers' bf16 outputs differ by their rounding (half a unit of bf16, 2^-9 of a value, plus fp32 sums:
6e-3 of the largest value), the per-channel fp32 results by fp32 sums (1e-5).
"""
import pytest
import torch

from test_gpu_parity import log

pytestmark = pytest.mark.gpu


def _close(got, want, tol):
    got, want = got.double(), want.double()
    assert torch.isfinite(got).all()
    assert float((got - want).abs().max()) <= tol * max(float(want.abs().max()), 1e-30)


@pytest.mark.parametrize("c", [1, 3, 7, 8, 19, 24, 100, 255, 256, 257, 2056])
@pytest.mark.parametrize("rows", [1, 2, 7, 8, 9, 15, 64, 333, 2051])
def test_batchnorm_layouts(tbn, rows, c):
    _layout(tbn, rows, c)


# the element-wise passes with one row and with four rows a thread (8 channels a thread: from 256 blocks of four on,
# one channel: from 768), the finalize with 16 and with 64 chunk lanes (from 209 chunks on), each with a last
# block that is partial
@pytest.mark.parametrize("rows,c", [(32640, 64), (32641, 64), (40000, 19), (39870, 19), (1021, 1024), (3333, 1024),
                                    (1999, 300), (1661, 1032), (1672, 1032)])
def test_batchnorm_rules(tbn, rows, c):
    _layout(tbn, rows, c)


def _layout(tbn, rows, c):
    log("batch normalisation %d x %d" % (rows, c))
    g = torch.Generator(device="cuda").manual_seed(rows * 4099 + c)
    x = (torch.randn(rows, c, generator=g, device="cuda") + torch.randn(c, generator=g, device="cuda")).bfloat16()
    dy = torch.randn(rows, c, generator=g, device="cuda").bfloat16()
    gamma = torch.rand(c, generator=g, device="cuda") + 0.5
    beta = torch.randn(c, generator=g, device="cuda")
    y, mean, inv = tbn.batchnorm_train_fwd(x, gamma, beta, relu=True)
    dx, dgamma, dbeta = tbn.batchnorm_train_bwd(x, y, dy, mean, inv, gamma, relu=True)
    again = tbn.batchnorm_train_bwd(x, y, dy, mean, inv, gamma, relu=True)
    xd, m = x.double(), x.double().mean(0)
    i = 1 / torch.sqrt(x.double().var(0, unbiased=False) + 1e-5)
    xh = (xd - m) * i
    _close(mean, m, 1e-5)
    _close(inv, i, 1e-5)
    _close(y, torch.relu(xh * gamma.double() + beta.double()), 6e-3)
    gd = torch.where(y.double() > 0, dy.double(), torch.zeros_like(xd))
    _close(dbeta, gd.sum(0), 1e-5)
    _close(dgamma, (gd * xh).sum(0), 1e-4 if rows == 2 else 1e-5)  # two rows: xh = +-1 up to the fp32 variance
    want = gamma.double() * i * (gd - gd.sum(0) / rows - xh * (gd * xh).sum(0) / rows)
    # the three terms cancel for few rows: the bound is on the terms, not on their difference
    scale = float((gamma.double() * i * gd).abs().max())
    assert float((dx.double() - want).abs().max()) <= 6e-3 * max(scale, 1e-30)
    assert all(torch.equal(s, t) for s, t in zip((dx, dgamma, dbeta), again))


@pytest.mark.parametrize("c", [1, 3, 7, 19, 100, 255])
def test_batchnorm_uneven_channels_of_a_large_tensor(tbn, c):
    rows = (1 << 21) // c + 8
    rows += (5 - rows) % 8  # a remainder of five rows against eight
    log("batch normalisation %d x %d" % (rows, c))
    g = torch.Generator(device="cuda").manual_seed(c)
    x = (torch.randn(rows, c, generator=g, device="cuda") + torch.randn(c, generator=g, device="cuda")).bfloat16()
    dy = torch.randn(rows, c, generator=g, device="cuda").bfloat16()
    gamma = torch.rand(c, generator=g, device="cuda") + 0.5
    beta = torch.randn(c, generator=g, device="cuda")
    y, mean, inv = tbn.batchnorm_train_fwd(x, gamma, beta, relu=True)
    dx, dgamma, dbeta = tbn.batchnorm_train_bwd(x, y, dy, mean, inv, gamma, relu=True)
    xd, m = x.double(), x.double().mean(0)
    i = 1 / torch.sqrt(x.double().var(0, unbiased=False) + 1e-5)
    xh = (xd - m) * i
    _close(mean, m, 1e-5)
    _close(inv, i, 1e-5)
    _close(y, torch.relu(xh * gamma.double() + beta.double()), 6e-3)
    gd = torch.where(y.double() > 0, dy.double(), torch.zeros_like(xd))
    # fp32 sums over up to about 1100 terms in a row: 2^-24 times that of the sum of the terms' sizes at worst
    for got, terms in ((dbeta, gd), (dgamma, gd * xh)):
        assert bool(((got.double() - terms.sum(0)).abs() <= 1100 * 2.0 ** -24 * terms.abs().sum(0)).all())
    want = gamma.double() * i * (gd - gd.mean(0) - xh * (gd * xh).mean(0))
    _close(dx, want, 6e-3)


@pytest.mark.parametrize("k", [2, 3])
@pytest.mark.parametrize("n,h,w,c", [(1, 2, 3, 8), (2, 7, 5, 16), (3, 9, 9, 24), (1, 4, 8, 40), (2, 6, 11, 5),
                                     (2, 126, 128, 32), (2, 127, 129, 32), (3, 115, 117, 56), (3, 115, 121, 56)])
def test_maxpool_backward_cells(tbn, k, n, h, w, c):
    if min(h, w) < k:
        pytest.skip("window larger than the input")
    log("pooling backward %s window %d" % ((n, h, w, c), k))
    g = torch.Generator(device="cuda").manual_seed(n * h * w * c + k)
    x = torch.relu(torch.randn(n, h, w, c, generator=g, device="cuda")).bfloat16()  # ties at zero
    y, arg = tbn.maxpool2d_fwd(x, k, k, 0, want_argmax=True)
    dy = torch.randn(y.shape, generator=g, device="cuda").bfloat16()
    want = torch.zeros(n, h * w, c, device="cuda")
    p, q = h // k, w // k
    want.scatter_(1, arg.view(n, p * q, c).long(), dy.float().view(n, p * q, c))
    for dtype in (torch.bfloat16, torch.float32):
        dx = tbn.maxpool2d_bwd(dy, arg, x.shape, k, k, 0, out_dtype=dtype)
        assert torch.equal(dx.float(), want.view(n, h, w, c))
