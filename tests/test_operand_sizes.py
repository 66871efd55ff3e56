"""Operands shorter than what the kernels read or write are refused before anything is queued: each call
with one operand a single element too short raises ValueError naming it, and a per-channel fp32 operand
given in 16 bits (half the bytes) raises TypeError.  On host tensors, whose device would be refused only
after the sizes, and on GPU tensors, where the native marshalling has to decline them.
"""
import pytest
import torch

import paper_1701_00485_amd as tbn_mod


def _calls(tbn, dev):
    def bf(*shape):
        return torch.zeros(shape, dtype=torch.bfloat16, device=dev)

    def f(*shape):
        return torch.zeros(shape, device=dev)

    def i(*shape):
        return torch.zeros(shape, dtype=torch.int32, device=dev)

    d = tbn.ConvDesc(2, 6, 5, 16, 24, 3, 3, 1, 1)
    x, w, codes, alpha, y = bf(2, 6, 5, 16), f(24, 3, 3, 16), i(64 * 3 * 4), f(24), bf(2, 6, 5, 24)
    stem = tbn.ConvDesc(64, 224, 224, 3, 64, 7, 7, 2, 3)
    sx, sc, sa = bf(1).expand(64, 224, 224, 3), i(64 * 3 * 4), f(64)
    calls = [
        ("counts", tbn.quantize, (w,), {"counts": i(47)}),
        ("counts", tbn.quantize_variant, (w, 0.5), {"counts": i(47)}),
        ("counts", tbn.sgd_step_quantize, (w, f(24, 144), f(24, 144), 0.1), {"counts": i(47)}),
        ("scale", tbn.conv2d_fwd, (d, x, codes, alpha), {"scale": f(23)}),
        ("bias", tbn.conv2d_fwd, (d, x, codes, alpha), {"bias": f(23)}),
        ("scale", tbn.conv2d_fwd_noalloc, (d, x, codes, alpha, y), {"scale": f(23)}),
        ("bias", tbn.conv2d_fwd_noalloc, (d, x, codes, alpha, y), {"bias": f(23)}),
        ("scale", tbn.conv2d_fwd_dense, (d, x, w), {"scale": f(23)}),
        ("bias", tbn.conv2d_fwd_dense, (d, x, w), {"bias": f(23)}),
        ("scale", tbn.conv2d_relu_maxpool_fwd, (stem, sx, sc, sa), {"scale": f(63)}),
        ("bias", tbn.conv2d_relu_maxpool_fwd, (stem, sx, sc, sa), {"bias": f(63)}),
        ("dy", tbn.maxpool2d_bwd, (bf(191), i(192), (2, 6, 5, 16), 2, 2, 0), {}),
        ("argmax", tbn.maxpool2d_bwd, (bf(192), i(191), (2, 6, 5, 16), 2, 2, 0), {}),
        ("gamma", tbn.batchnorm_train_fwd, (x, f(15), f(16)), {}),
        ("beta", tbn.batchnorm_train_fwd, (x, f(16), f(15)), {}),
        ("y", tbn.relu_bwd, (bf(959), x), {}),
        ("labels", tbn.softmax_xent, (f(5, 10), i(4)), {}),
    ]
    bn = {"x": x, "y": x, "dy": x, "mean": f(16), "inv_std": f(16), "gamma": f(16)}
    for name in ("y", "dy", "mean", "inv_std", "gamma"):
        short = torch.zeros(bn[name].numel() - 1, dtype=bn[name].dtype, device=dev)
        calls.append((name, tbn.batchnorm_train_bwd, (), dict(bn, **{name: short})))
    return calls, bn


def _check(tbn, dev):
    calls, bn = _calls(tbn, dev)
    for name, call, args, kw in calls:
        print(call.__name__, name, flush=True)
        with pytest.raises(ValueError, match="^%s has" % name):
            call(*args, **kw)
    return bn


def test_short_operands_of_host_tensors():
    _check(tbn_mod, "cpu")


@pytest.mark.gpu
def test_short_operands_of_gpu_tensors(tbn):
    bn = _check(tbn, "cuda")
    half = torch.zeros(16, dtype=torch.bfloat16, device="cuda")
    for name in ("mean", "inv_std", "gamma", "dgamma", "dbeta"):
        print("batchnorm_train_bwd 16-bit", name, flush=True)
        with pytest.raises(TypeError, match="^%s has dtype" % name):
            tbn.batchnorm_train_bwd(**dict(bn, **{name: half}))
