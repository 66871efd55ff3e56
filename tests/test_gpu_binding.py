"""The native marshalling of the Python calls: every call gives bit for bit what the ctypes code
gives for the same arguments (allocated and caller-provided outputs, optional operands given and
not), and what it declines raises what the ctypes code raises.  That it answers the ordinary calls itself and
declines the others is recorded: where it declined everything, both sides would run the ctypes code.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


class _Declines:
    """Stands in for the native module: declines every call."""

    def __getattr__(self, name):
        return lambda *args: NotImplemented


LIBRARY_REFUSES = ("small workspace", "misaligned", "stride")


def _tensors(o):
    if isinstance(o, torch.Tensor):
        return [o.clone()]
    return [] if o is None else [t for x in o for t in _tensors(x)]


def _calls(tbn):
    g = torch.Generator(device="cuda").manual_seed(7)

    def rnd(*shape, dtype=torch.float32):
        return torch.randn(shape, generator=g, device="cuda").to(dtype)

    bf = torch.bfloat16
    d = tbn.ConvDesc(2, 6, 5, 16, 24, 3, 3, 1, 1)
    x, dy, w = rnd(2, 6, 5, 16, dtype=bf), rnd(2, 6, 5, 24, dtype=bf), rnd(24, 3, 3, 16)
    codes, alpha, _ = tbn.quantize(w)
    vec, res = rnd(24), rnd(2, 6, 5, 24, dtype=bf)
    ws = tbn.workspace(tbn.OP_BWD_DATA, d)
    q8, f8 = tbn.quantize_act_i8(x, 20.0), tbn.quantize_act_fp8(x, 20.0)
    fp4 = tbn.repack_codes_fp4(codes)
    gamma, beta = rnd(16), rnd(16)
    a, mean, inv = tbn.batchnorm_train_fwd(x, gamma, beta, relu=True)
    p, arg = tbn.maxpool2d_fwd(x, 2, 2, 0, want_argmax=True)
    logits, labels = rnd(5, 10), torch.arange(5, device="cuda", dtype=torch.int32)
    return {
        "quantize": lambda: tbn.quantize(w),
        "quantize no counts": lambda: tbn.quantize(w, codes=torch.empty_like(codes), want_counts=False),
        "quantize counts": lambda: tbn.quantize(w, counts=torch.empty(24, 2, dtype=torch.int32, device="cuda"),
                                                want_counts=False),
        "fwd": lambda: tbn.conv2d_fwd(d, x, codes, alpha),
        "fwd epilogue": lambda: tbn.conv2d_fwd(d, x, codes, alpha, scale=vec, bias=vec, residual=res, relu=True),
        "fwd fp32 in and out": lambda: tbn.conv2d_fwd(d, x.float(), codes, alpha, out_dtype=torch.float32, bias=vec),
        "fwd y": lambda: tbn.conv2d_fwd(d, x, codes, alpha, y=torch.empty(2, 6, 5, 24, device="cuda"), relu=True),
        "dense": lambda: tbn.conv2d_fwd_dense(d, x, w, bias=vec),
        "i8": lambda: tbn.conv2d_fwd_i8(d, q8, codes, alpha, 0.05, relu=True),
        "fp8": lambda: tbn.conv2d_fwd_fp8(d, f8, fp4, alpha, 0.05, out_dtype=torch.float32),
        "bwd_data": lambda: tbn.conv2d_bwd_data(d, dy, codes, alpha),
        "bwd_data ws": lambda: tbn.conv2d_bwd_data(d, dy, codes, alpha, out_dtype=torch.float32, ws=ws),
        "bwd_weight": lambda: tbn.conv2d_bwd_weight(d, x, dy),
        "bwd_weight add": lambda: tbn.conv2d_bwd_weight(d, x, dy, dw=w.clone(), accumulate=True),
        "sgd": lambda: tbn.sgd_step(w.clone(), torch.zeros_like(w), w, 0.1),
        "sgd quantize": lambda: tbn.sgd_step_quantize(w.clone(), torch.zeros_like(w), w, 0.1, 0.5, 0),
        "act i8": lambda: tbn.quantize_act_i8(x, 20.0),
        "act fp8": lambda: tbn.quantize_act_fp8(x.float(), 20.0),
        "maxpool": lambda: tbn.maxpool2d_fwd(x, 3, 2, 1, want_argmax=True),
        "maxpool y": lambda: tbn.maxpool2d_fwd(x, 2, 2, 0),
        "maxpool bwd": lambda: tbn.maxpool2d_bwd(p, arg, x.shape, 2, 2, 0, out_dtype=torch.float32),
        "avgpool": lambda: tbn.avgpool_global(x, out_dtype=torch.float32),
        "bn": lambda: tbn.batchnorm_train_fwd(x, gamma, beta),
        "bn bwd": lambda: tbn.batchnorm_train_bwd(x, a, x, mean, inv, gamma, relu=True, dgamma=torch.empty_like(gamma)),
        "relu bwd": lambda: tbn.relu_bwd(x, a),
        "xent": lambda: tbn.softmax_xent(logits, labels),
    }, {
        # declined: the errors are those of the ctypes code
        "cpu tensor": lambda: tbn.relu_bwd(x.cpu(), x),
        "strided": lambda: tbn.conv2d_fwd(d, x.transpose(1, 2), codes, alpha),
        "size": lambda: tbn.conv2d_fwd(d, x[:1], codes, alpha),
        "type": lambda: tbn.conv2d_bwd_weight(d, x.float(), dy),
        "residual type": lambda: tbn.conv2d_fwd(d, x, codes, alpha, residual=res.float()),
        "small workspace": lambda: tbn.conv2d_bwd_data(d, dy, codes, alpha, ws=torch.empty(16, device="cuda")),
        "misaligned": lambda: tbn.conv2d_fwd(d, torch.empty(x.numel() + 1, dtype=bf, device="cuda")[1:], codes, alpha),
        "stride": lambda: tbn.conv2d_bwd_data(tbn.ConvDesc(2, 6, 5, 16, 24, 3, 3, 2, 1), dy[:, :3, :3].contiguous(),
                                              codes, alpha),
        "geometry": lambda: tbn.conv2d_fwd(tbn.ConvDesc(2, 6, 5, 16, 24, 9, 9, 1, 0), x, codes, alpha),
    }


class _Recorder:
    """Passes calls on to the native module and notes which of them it declined."""

    def __init__(self, module):
        self.module, self.answered, self.declined = module, 0, 0

    def __getattr__(self, name):
        def call(*args):
            try:
                out = getattr(self.module, name)(*args)
            except Exception:  # an error of the library: the call was taken
                self.answered += 1
                raise
            self.declined += out is NotImplemented
            self.answered += out is not NotImplemented
            return out
        return call


def test_native_calls_equal_ctypes_calls(tbn, monkeypatch):
    ordinary, refused = _calls(tbn)
    monkeypatch.setattr(tbn, "_native", None)

    def outcome(f):
        try:
            return _tensors(f())
        except Exception as e:  # the type and the message are compared
            return (type(e), str(e))

    native, module = {}, tbn._load_native()
    for calls in (ordinary, refused):
        for name, f in calls.items():
            recorder = _Recorder(module)
            monkeypatch.setattr(tbn, "_native", recorder)
            native[name] = outcome(f)
            took = (recorder.answered, recorder.declined)
            # what the library itself refuses (alignment, workspace, stride) is still an ordinary call to the binding
            assert took == ((1, 0) if calls is ordinary or name in LIBRARY_REFUSES else (0, 1)), (name, took)
    monkeypatch.setattr(tbn, "_native", _Declines())
    for name, f in list(ordinary.items()) + list(refused.items()):
        print(name, flush=True)
        got, want = native[name], outcome(f)
        if name in refused:
            assert isinstance(want, tuple) and got == want
            continue
        assert not isinstance(got, tuple), got
        assert [(t.shape, t.dtype) for t in got] == [(t.shape, t.dtype) for t in want]
        assert all(torch.equal(s, t) for s, t in zip(got, want))
