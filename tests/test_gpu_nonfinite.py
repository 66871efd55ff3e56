"""Infinities and NaN in the inputs of the kernels that read past an image, a filter, a split or the real
channels into padding: they reach exactly the outputs whose windows hold them (padding is multiplied as
zero, and never by a neighbour's infinity), every other output has the bits that it has with zeros in
their place, and ReLU takes NaN to zero as it does everywhere.  Shapes: small-layer kernel, 64-channel kernel, tiled
kernel, general kernel, channel-padded copies with odd counts; both passes; narrow and wide
filter-gradient tiles, the register-staged kernel.  The pattern is torch's on the CPU in fp64 with the decoded
codes; where a window holds infinities of both signs or a NaN the result is NaN.
"""
import pytest
import torch
import torch.nn.functional as F

from test_gpu_parity import log

pytestmark = pytest.mark.gpu

# n, h, w, c, k, r, pad, forward tile (small layers 51-55, 64 channels 60, tiled 14 and 18, general 0)
CASES = [(1, 5, 7, 24, 66, 3, 1, 51), (2, 5, 7, 72, 40, 3, 1, 53), (1, 6, 6, 128, 96, 3, 1, 55), (2, 6, 11, 64, 40, 3, 1, 60),
         (2, 9, 13, 40, 72, 3, 1, 14), (2, 9, 13, 128, 130, 3, 1, 18), (2, 5, 6, 12, 20, 3, 1, 0), (2, 5, 6, 13, 21, 3, 1, -1),
         (1, 4, 5, 65, 9, 3, 1, -1), (2, 7, 5, 9, 33, 5, 2, -1)]


def _special(t, g, count):
    """The tensor with infinities of both signs and NaN at random places, and with zeros there."""
    flat = t.reshape(-1)
    at = torch.randperm(flat.numel(), generator=g)[:count]
    values = torch.tensor([float("inf"), float("-inf"), float("nan")]).repeat(count)[:count]
    odd, zero = flat.clone(), flat.clone()
    odd[at], zero[at] = values.to(t.dtype), 0
    return odd.reshape(t.shape).cuda(), zero.reshape(t.shape).cuda()


def _levels(w):
    a = w.abs().mean(1, keepdim=True)
    return torch.where(w >= 0, 1.0, -1.0) * torch.where(w.abs() > a, 2.0, 1.0)


def _same(got, clean, pattern):
    """Non-finite where `pattern` is, the same infinities, and the bits of `clean` elsewhere."""
    got, clean, pattern = got.float().cpu(), clean.float().cpu(), pattern.float()
    hit = ~torch.isfinite(pattern)
    assert bool(hit.any()) and not bool(hit.all())
    assert torch.equal(torch.isnan(got), torch.isnan(pattern))
    assert torch.equal(torch.isinf(got), torch.isinf(pattern))
    inf = torch.isinf(pattern)
    assert torch.equal(got[inf], pattern[inf])
    assert torch.equal(got[~hit], clean[~hit])


@pytest.mark.parametrize("case", CASES, ids=str)
def test_nonfinite_inputs(tbn, case, knobs):
    n, h, w, c, k, r, pad, tile = case
    g = torch.Generator().manual_seed(n * h * w * c * k)
    d = tbn.ConvDesc(n, h, w, c, k, r, r, 1, pad)
    p, q = d.out_dims()
    wt = torch.randn(k, r * r * c, generator=g)
    codes, alpha, _ = tbn.quantize(wt.cuda())
    lv = _levels(wt).view(k, r, r, c).permute(0, 3, 1, 2).double()
    x, xz = _special(torch.randn(n, h, w, c, generator=g).bfloat16(), g, 3)
    dy, dyz = _special(torch.randn(n, p, q, k, generator=g).bfloat16(), g, 3)
    nchw = lambda t: t.cpu().double().permute(0, 3, 1, 2)

    log("non-finite inputs forward %s" % (case,))
    knobs(conv_tile=tile)
    want = F.conv2d(nchw(x), lv, padding=pad).permute(0, 2, 3, 1)
    _same(tbn.conv2d_fwd(d, x, codes, alpha), tbn.conv2d_fwd(d, xz, codes, alpha), want)
    y, yz = (tbn.conv2d_fwd(d, t, codes, alpha, relu=True).float().cpu() for t in (x, xz))
    hit = ~torch.isfinite(want)
    assert torch.equal(y[~hit], yz[~hit])
    assert torch.equal(y[hit], torch.where(want[hit] > 0, want[hit], torch.zeros(())).float())  # NaN: 0

    log("non-finite gradient backward-data %s" % (case,))
    knobs(conv_tile=-1)
    want = F.conv_transpose2d(nchw(dy), lv, padding=pad).permute(0, 2, 3, 1)
    _same(tbn.conv2d_bwd_data(d, dy, codes, alpha), tbn.conv2d_bwd_data(d, dyz, codes, alpha), want)

    # filter gradient: non-finite activations, so that what padding multiplies is finite
    taps = F.pad(nchw(x), (pad, pad, pad, pad))
    want = torch.zeros(k, r, r, c, dtype=torch.float64)
    gy = dyz.cpu().double().reshape(-1, k)
    for i in range(r):
        for j in range(r):
            want[:, i, j] = gy.t() @ taps[:, :, i:i + p, j:j + q].permute(0, 2, 3, 1).reshape(-1, c)
    for cfg in (-1, 0, 1):
        log("non-finite activations filter gradient %s kernel %d" % (case, cfg))
        knobs(wgrad_cfg=cfg)
        _same(tbn.conv2d_bwd_weight(d, x, dyz), tbn.conv2d_bwd_weight(d, xz, dyz), want)
    if c % 8 and k % 8:
        log("non-finite activations filter gradient %s without workspace for copies" % (case,))
        ws = torch.empty(16, dtype=torch.uint8, device="cuda")
        _same(tbn.conv2d_bwd_weight(d, x, dyz, ws=ws), tbn.conv2d_bwd_weight(d, xz, dyz, ws=ws), want)
