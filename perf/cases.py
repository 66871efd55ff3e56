"""The work that users of the package have it do, as cases to time and to compare.

Every case goes through the public calls of ``paper_1701_00485_amd`` (and ``networks``) the way
the training loops and the inference network of this repository do: outputs allocated by the
call, workspace left to it, one stream.  Inputs are drawn on the GPU from the seed alone.

Kinds of case (field "kind"):
  first   a first layer: few input channels, fp32 or bf16 images, forward (the single 5x5
          layer on 28 x 28 digits, LeNet's first layer, the 7x7 RGB stem)
  train   one two-bit layer's share of a training iteration (Algorithm 1): forward, gradient to
          the input, straight-through gradient to the real filters, update -- with the
          quantisation in front (`fused` false) or fused into the update (`fused` true)
  glue    what stands between two convolutions of a training network, forward and backward:
          batch normalisation + ReLU (`bn`) or ReLU alone, and max pooling (`pool` 2: 2x2/2,
          3: 3x3/2 pad 1, 0: none)
  head    the classifier of a training network: logits, softmax cross-entropy, both gradients
  block   a residual block at inference (two 3x3 convolutions with folded batch normalisation,
          the shortcut and the projection where the shape changes)
  fc      a fully-connected layer at inference (weight streaming at small batches)
  i8/fp8  the low-precision forward pass: activation codes, then the convolution on them
  resnet  the whole ResNet-18 forward, images to logits
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

import paper_1701_00485_amd as tbn
from paper_1701_00485_amd import networks

LR, MU, WD = 0.1, 0.9, 1e-4


# ------------------------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest call: one 5x5 layer on 16 digits, fp32 pixels; launch latency counts
        {"name": "first_5x5_n16", "kind": "first", "n": 16, "h": 28, "w": 28, "c": 1, "k": 32, "r": 5, "stride": 1,
         "pad": 2, "f32": True},
        # one image through the whole network, as a server answers one request
        {"name": "resnet18_n1", "kind": "resnet", "n": 1, "h": 224, "w": 224},
        # a batch of images through the whole network
        {"name": "resnet18_n64", "kind": "resnet", "n": 64, "h": 224, "w": 224},
        # the block where the resolution halves (strided 3x3, 1x1 projection), a batch that is no power of two
        {"name": "block_64_128_n24", "kind": "block", "n": 24, "h": 56, "w": 56, "c": 64, "k": 128, "stride": 2},
        # the large training layer, quantised, run both ways and updated
        {"name": "train_3x3_256_n128", "kind": "train", "n": 128, "h": 56, "w": 56, "c": 256, "k": 256, "r": 3,
         "pad": 1, "fused": False},
        # LeNet's second layer with the fused update
        {"name": "train_5x5_64_n256", "kind": "train", "n": 256, "h": 14, "w": 14, "c": 32, "k": 64, "r": 5, "pad": 2,
         "fused": True},
        # a training layer whose sizes fit no tile: odd map, odd batch, channel counts that are no multiple of 8
        {"name": "train_3x3_ragged", "kind": "train", "n": 50, "h": 27, "w": 19, "c": 36, "k": 100, "r": 3, "pad": 1,
         "fused": True},
        # after VGG-small's second convolution: normalise, ReLU, pool, and back
        {"name": "glue_32x32x128_n128", "kind": "glue", "n": 128, "h": 32, "w": 32, "c": 128, "bn": True, "pool": 2},
        # VGG-small's classifier in training (8192 -> 10 as a 4x4 window)
        {"name": "head_8192_10_n128", "kind": "head", "n": 128, "h": 4, "c": 512, "k": 10},
        # a large fully-connected layer for one input: bound by streaming its codes
        {"name": "fc_8192_32768_n1", "kind": "fc", "n": 1, "c": 8192, "k": 32768},
        # low-precision inference, a middle and a large layer
        {"name": "i8_28x28_128_n64", "kind": "i8", "n": 64, "h": 28, "w": 28, "c": 128, "k": 128, "r": 3},
        {"name": "fp8_56x56_256_n32", "kind": "fp8", "n": 32, "h": 56, "w": 56, "c": 256, "k": 256, "r": 3},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi, step=1):
    """Mostly multiples of 8, as networks have; one in four as it falls."""
    c = _log(rng, lo, hi)
    step = max(step, 8 if rng.random() < 0.75 else 1)
    return max(step, (c + step // 2) // step * step)


def _map(rng, lo, hi):
    """Height and width of a feature map: square half the time, else nearly so."""
    h = _log(rng, lo, hi)
    return h, max(lo, h + rng.choice([0, 0, 0, -1, 3, h // 2]))


def _fit(case, most_flops, most_bytes):
    """The batch lowered until the case costs no more than allowed."""
    while case["n"] > 1:
        w = work(case)
        if w["flops"] <= most_flops and w["bytes"] <= most_bytes:
            break
        case["n"] = max(1, min(case["n"] - 1, int(case["n"] * 0.8)))
    return case


def draw(rng):
    kind = rng.choice(["first", "train", "train", "glue", "head", "block", "fc", "i8", "fp8", "resnet"])
    if kind == "first":
        c = rng.choice([1, 1, 3, 3, 4])
        r, stride = rng.choice([(3, 1), (5, 1), (7, 2)])
        h, w = _map(rng, 24, 224)
        return _fit({"kind": kind, "n": _log(rng, 1, 256), "h": h, "w": w, "c": c, "k": _channels(rng, 16, 128), "r": r,
                     "stride": stride, "pad": r // 2, "f32": rng.random() < 0.5}, 2e10, 3e8)
    if kind == "train":
        c, k = _channels(rng, 1, 512), _channels(rng, 8, 512)
        r = rng.choice([1, 3, 3, 3, 5])
        most = 7e11 if c % 8 == 0 else 2e10
        h, w = _map(rng, 7, 56)
        return _fit({"kind": kind, "n": _log(rng, 4, 256), "h": h, "w": w, "c": c, "k": k, "r": r, "pad": r // 2,
                     "fused": rng.random() < 0.5}, most, 8e8)
    if kind == "glue":
        h, w = _map(rng, 7, 112)
        return _fit({"kind": kind, "n": _log(rng, 4, 256), "h": h, "w": w, "c": _channels(rng, 16, 512),
                     "bn": rng.random() < 0.75, "pool": rng.choice([0, 2, 2, 3])}, 1e30, 8e8)
    if kind == "head":
        return {"kind": kind, "n": _log(rng, 8, 512), "h": rng.choice([1, 1, 4, 7]), "c": _channels(rng, 64, 512, 8),
                "k": _log(rng, 2, 1000)}
    if kind == "block":
        stride = rng.choice([1, 1, 2])
        c = _channels(rng, 32, 512, 8)
        h, w = _map(rng, 7, 56)
        return _fit({"kind": kind, "n": _log(rng, 1, 64), "h": h, "w": w, "c": c,
                     "k": c if stride == 1 else min(512, 2 * c), "stride": stride}, 2e11, 4e8)
    if kind == "fc":
        return {"kind": kind, "n": _log(rng, 1, 64), "c": _channels(rng, 256, 16384, 8),
                "k": _channels(rng, 100, 32768)}
    if kind in ("i8", "fp8"):
        h, w = _map(rng, 7, 56)
        return _fit({"kind": kind, "n": _log(rng, 1, 128), "h": h, "w": w, "c": _channels(rng, 32, 512, 16),
                     "k": _channels(rng, 32, 512), "r": rng.choice([1, 3, 3])}, 4e11, 6e8)
    return {"kind": "resnet", "n": _log(rng, 1, 64), "h": rng.choice([160, 192, 224, 224, 225]),
            "w": rng.choice([160, 192, 224, 224, 251])}


def _out(case):
    r, s, p = case.get("r", 3), case.get("stride", 1), case.get("pad", case.get("r", 3) // 2)
    return (case["h"] + 2 * p - r) // s + 1, (case["w"] + 2 * p - r) // s + 1


def _pooled(case):
    h, w = case["h"], case["w"]
    return {0: (h, w), 2: (h // 2, w // 2), 3: ((h - 1) // 2 + 1, (w - 1) // 2 + 1)}[case["pool"]]


def _resnet_layers(case):
    """(name, cin, cout, k, stride, pad, h, w of the input) of every convolution but the classifier."""
    h, w = case["h"], case["w"]
    out = [("stem", 3, 64, 7, 2, 3, h, w)]
    h, w = (h - 1) // 2 + 1, (w - 1) // 2 + 1
    h, w = (h - 1) // 2 + 1, (w - 1) // 2 + 1
    cin = 64
    for i, (cout, stride) in enumerate([(64, 1), (128, 2), (256, 2), (512, 2)]):
        for j in range(2):
            s = stride if j == 0 else 1
            name = "layer%d.%d" % (i + 1, j)
            ho, wo = (h - 1) // s + 1, (w - 1) // s + 1
            out.append((name + ".conv1", cin, cout, 3, s, 1, h, w))
            if s != 1 or cin != cout:
                out.append((name + ".downsample", cin, cout, 1, s, 0, h, w))
            out.append((name + ".conv2", cout, cout, 3, 1, 1, ho, wo))
            h, w, cin = ho, wo, cout
    return out


def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "first":
        p, q = _out(case)
        m, e = n * p * q, case["r"] ** 2 * case["c"]
        return {"bytes": n * case["h"] * case["w"] * case["c"] * (4 if case["f32"] else 2) + m * case["k"] * 2 +
                case["k"] * e / 4 + case["k"] * 4, "flops": 2 * m * case["k"] * e}
    if kind == "train":
        p, q = _out(case)
        m, e = n * p * q, case["r"] ** 2 * case["c"]
        act = n * case["h"] * case["w"] * case["c"] * 2
        dx = case["c"] >= 8  # a first layer needs no input gradient
        return {"bytes": act * (2 if dx else 1) + 2 * m * case["k"] * 2 + case["k"] * e * (4 * 5 + 0.25) +
                case["k"] * 4, "flops": (6 if dx else 4) * m * case["k"] * e}
    if kind == "glue":
        full = n * case["h"] * case["w"] * case["c"]
        p, q = _pooled(case)
        small = n * p * q * case["c"]
        b = 2 * full + 2 * full + 2 * full  # x in, activation out, dx out
        b += (2 + 4 + 2) * small if case["pool"] else 2 * full  # pooled out, argmax out, dy in (or dy in)
        return {"bytes": b, "flops": 20 * full}
    if kind == "head":
        e = case["h"] ** 2 * case["c"]
        return {"bytes": n * e * 4 + case["k"] * e * 4.25 + n * case["k"] * 6 + n * 4, "flops": 6 * n * case["k"] * e}
    if kind == "block":
        p, q = _out(case)
        m = n * p * q
        e = 9 * case["c"] + 9 * case["k"] + (case["c"] if case["stride"] != 1 else 0)
        return {"bytes": n * case["h"] * case["w"] * case["c"] * 2 + m * case["k"] * 2 + case["k"] * e / 4,
                "flops": 2 * m * case["k"] * e}
    if kind == "fc":
        return {"bytes": case["c"] * case["k"] / 4 + n * (2 * case["c"] + 2 * case["k"]) + 4 * case["k"],
                "flops": 2 * n * case["c"] * case["k"]}
    if kind in ("i8", "fp8"):
        p, q = _out(case)
        m, e = n * p * q, case["r"] ** 2 * case["c"]
        return {"bytes": n * case["h"] * case["w"] * case["c"] * 3 + m * case["k"] * 2 + case["k"] * e / 4,
                "flops": 2 * m * case["k"] * e}
    flops, codes = 2 * n * 512 * 1000, 512 * 1000
    for _, cin, cout, k, s, p, h, w in _resnet_layers(case):
        ho, wo = (h + 2 * p - k) // s + 1, (w + 2 * p - k) // s + 1
        flops += 2 * n * ho * wo * cout * k * k * cin
        codes += k * k * cin * cout
    return {"bytes": n * case["h"] * case["w"] * 3 * 2 + codes / 4 + n * 4000, "flops": flops}


# ------------------------------------------------------------------------------------ inputs
class _Draws:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)

    def normal(self, *shape, std=1.0, mean=0.0, dtype=torch.bfloat16):
        return (torch.randn(shape, generator=self.g, device="cuda") * std + mean).to(dtype)

    def uniform(self, *shape, lo=0.0, hi=1.0, dtype=torch.float32):
        return (torch.rand(shape, generator=self.g, device="cuda") * (hi - lo) + lo).to(dtype)

    def labels(self, n, k):
        return torch.randint(0, k, (n,), generator=self.g, device="cuda", dtype=torch.int32)

    def folded_bn(self, k):
        """Scale and bias of a batch normalisation folded into the convolution before it."""
        scale = self.uniform(k, lo=0.5, hi=1.5) / torch.sqrt(self.uniform(k, lo=0.5, hi=1.5) + 1e-5)
        beta, mean = (self.normal(k, std=0.1, dtype=torch.float32) for _ in range(2))
        return scale, beta - mean * scale


def _inputs(case, seed):
    d, kind, n = _Draws(seed), case["kind"], case["n"]
    if kind == "first":
        dtype = torch.float32 if case["f32"] else torch.bfloat16
        return {"x": d.uniform(n, case["h"], case["w"], case["c"], dtype=dtype),
                "w": d.normal(case["k"], case["r"] ** 2 * case["c"], std=0.05, dtype=torch.float32)}
    if kind == "train":
        p, q = _out(case)
        # activations after a ReLU are half zeros; the gradient is of a mean over the batch, so that
        # the filter gradient is small against the filters
        return {"x": torch.relu(d.normal(n, case["h"], case["w"], case["c"])),
                "dy": d.normal(n, p, q, case["k"], std=0.01 / math.sqrt(n * p * q)),
                "w": d.normal(case["k"], case["r"] ** 2 * case["c"], std=0.05, dtype=torch.float32)}
    if kind == "glue":
        p, q = _pooled(case)
        c = case["c"]
        x = d.normal(n, case["h"], case["w"], c) + d.normal(c)
        return {"x": x if case["bn"] else torch.relu(x), "dy": d.normal(n, p, q, c, std=1e-2),
                "gamma": d.uniform(c, lo=0.5, hi=1.5), "beta": d.normal(c, std=0.1, dtype=torch.float32)}
    if kind == "head":
        return {"x": torch.relu(d.normal(n, case["h"], case["h"], case["c"])), "labels": d.labels(n, case["k"]),
                "w": d.normal(case["k"], case["h"] ** 2 * case["c"], std=0.05, dtype=torch.float32)}
    if kind == "block":
        c, k = case["c"], case["k"]
        t = {"x": torch.relu(d.normal(n, case["h"], case["w"], c))}
        for name, e in (("1", 9 * c), ("2", 9 * k)) + ((("d", c),) if case["stride"] != 1 else ()):
            t["w" + name] = d.normal(k, e, std=math.sqrt(2.0 / e), dtype=torch.float32)
            t["scale" + name], t["bias" + name] = d.folded_bn(k)
        return t
    if kind == "fc":
        return {"x": torch.relu(d.normal(n, 1, 1, case["c"])),
                "w": d.normal(case["k"], case["c"], std=math.sqrt(2.0 / case["c"]), dtype=torch.float32),
                "bias": d.normal(case["k"], std=0.01, dtype=torch.float32)}
    if kind in ("i8", "fp8"):
        e = case["r"] ** 2 * case["c"]
        x = torch.relu(d.normal(n, case["h"], case["w"], case["c"]))
        # the scale of a calibrated model: fixed, a little below the largest value
        return {"x": x, "scale": float(np.float32(4.5 / (127.0 if kind == "i8" else 448.0))),
                "w": d.normal(case["k"], e, std=math.sqrt(2.0 / e), dtype=torch.float32)}
    t = {"x": d.normal(n, case["h"], case["w"], 3)}
    for name, cin, cout, k, *_ in _resnet_layers(case):
        e = k * k * cin
        t[name] = (d.normal(cout, e, std=math.sqrt(2.0 / e), dtype=torch.float32),) + d.folded_bn(cout)
    t["fc"] = (d.normal(1000, 512, std=math.sqrt(2.0 / 512), dtype=torch.float32), None,
               d.normal(1000, std=0.01, dtype=torch.float32))
    return t


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case)
    kind, n = case["kind"], case["n"]
    if kind == "first":
        s["desc"] = tbn.ConvDesc(n, case["h"], case["w"], case["c"], case["k"], case["r"], case["r"], case["stride"],
                                 case["pad"])
        s["codes"], s["alpha"], _ = tbn.quantize(s["w"], want_counts=False)
    elif kind == "train":
        s["desc"] = tbn.ConvDesc(n, case["h"], case["w"], case["c"], case["k"], case["r"], case["r"], 1, case["pad"])
        s["v"] = torch.zeros_like(s["w"])
        s["codes"], s["alpha"], _ = tbn.quantize(s["w"], want_counts=False)
    elif kind == "head":
        s["desc"] = tbn.ConvDesc(n, case["h"], case["h"], case["c"], case["k"], case["h"], case["h"], 1, 0)
        s["codes"], s["alpha"], _ = tbn.quantize(s["w"], want_counts=False)
    elif kind == "block":
        c, k, st = case["c"], case["k"], case["stride"]
        p, q = _out(case)
        s["desc1"] = tbn.ConvDesc(n, case["h"], case["w"], c, k, 3, 3, st, 1)
        s["desc2"] = tbn.ConvDesc(n, p, q, k, k, 3, 3, 1, 1)
        s["descd"] = tbn.ConvDesc(n, case["h"], case["w"], c, k, 1, 1, st, 0)
        for name in ("1", "2") + (("d",) if st != 1 else ()):
            s["codes" + name], s["alpha" + name], _ = tbn.quantize(s["w" + name], want_counts=False)
    elif kind == "fc":
        s["desc"] = tbn.ConvDesc(n, 1, 1, case["c"], case["k"], 1, 1, 1, 0)
        s["codes"], s["alpha"], _ = tbn.quantize(s["w"], want_counts=False)
        del s["w"]
    elif kind in ("i8", "fp8"):
        s["desc"] = tbn.ConvDesc(n, case["h"], case["w"], case["c"], case["k"], case["r"], case["r"], 1, case["r"] // 2)
        s["codes"], s["alpha"], _ = tbn.quantize(s["w"], want_counts=False)
        if kind == "fp8":
            s["codes"] = tbn.repack_codes_fp4(s["codes"])
    elif kind == "resnet":
        # the network object with these weights loaded into it
        net = networks.ResNet18.__new__(networks.ResNet18)
        net.device, net.classes = "cuda", 1000

        def layer(name, cin, cout, k, stride, pad):
            conv = networks.Conv.__new__(networks.Conv)
            conv.name, conv.cin, conv.cout, conv.k, conv.stride, conv.pad = name, cin, cout, k, stride, pad
            w, conv.scale, conv.bias = s[name]
            conv.codes, conv.alpha, _ = tbn.quantize(w, want_counts=False)
            return conv

        convs = {a[0]: layer(*a[:6]) for a in _resnet_layers(case)}
        net.stem = convs["stem"]
        net.blocks = [(convs[b + ".conv1"], convs[b + ".conv2"], convs.get(b + ".downsample"))
                      for b in ("layer%d.%d" % (i, j) for i in (1, 2, 3, 4) for j in (0, 1))]
        net.fc = layer("fc", 512, 1000, 1, 1, 0)
        s = {"case": case, "x": s["x"], "net": net}
    return s


# --------------------------------------------------------------------------------- the calls
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "first":
        return tbn.conv2d_fwd(s["desc"], s["x"], s["codes"], s["alpha"])
    if kind == "train":
        d = s["desc"]
        if not case["fused"]:
            tbn.quantize(s["w"], codes=s["codes"], alpha=s["alpha"], want_counts=False)
        y = tbn.conv2d_fwd(d, s["x"], s["codes"], s["alpha"])
        dx = tbn.conv2d_bwd_data(d, s["dy"], s["codes"], s["alpha"]) if case["c"] >= 8 else None
        dw = tbn.conv2d_bwd_weight(d, s["x"], s["dy"])
        if case["fused"]:
            tbn.sgd_step_quantize(s["w"], s["v"], dw.view(s["w"].shape), LR, MU, WD, codes=s["codes"], alpha=s["alpha"],
                                  want_counts=False)
        else:
            tbn.sgd_step(s["w"], s["v"], dw.view(s["w"].shape), LR, MU, WD)
        return {"y": y, "dx": dx, "dw": dw, "w": s["w"], "v": s["v"], "codes": s["codes"], "alpha": s["alpha"]}
    if kind == "glue":
        x, out = s["x"], {}
        if case["bn"]:
            a, mean, inv = tbn.batchnorm_train_fwd(x, s["gamma"], s["beta"], relu=True)
            out.update(a=a, mean=mean, inv=inv)
        else:
            a = x  # the convolution before it has applied the ReLU
        k, st, pad = {0: (0, 0, 0), 2: (2, 2, 0), 3: (3, 2, 1)}[case["pool"]]
        da = s["dy"]
        if k:
            out["p"], out["arg"] = tbn.maxpool2d_fwd(a, k, st, pad, want_argmax=True)
            da = tbn.maxpool2d_bwd(s["dy"], out["arg"], a.shape, k, st, pad)
        if case["bn"]:
            out["dx"], out["dgamma"], out["dbeta"] = tbn.batchnorm_train_bwd(x, a, da, mean, inv, s["gamma"], relu=True)
        else:
            out["dx"] = tbn.relu_bwd(a, da)
        return out
    if kind == "head":
        d, n, k = s["desc"], case["n"], case["k"]
        z = tbn.conv2d_fwd(d, s["x"], s["codes"], s["alpha"], out_dtype=torch.float32)
        loss, dz = tbn.softmax_xent(z.view(n, k), s["labels"])
        dz = dz.view(n, 1, 1, k)
        dx = tbn.conv2d_bwd_data(d, dz, s["codes"], s["alpha"])
        return {"z": z, "loss": loss, "dz": dz, "dx": dx, "dw": tbn.conv2d_bwd_weight(d, s["x"], dz)}
    if kind == "block":
        x = s["x"]
        a = tbn.conv2d_fwd(s["desc1"], x, s["codes1"], s["alpha1"], scale=s["scale1"], bias=s["bias1"], relu=True)
        sc = x if case["stride"] == 1 else tbn.conv2d_fwd(s["descd"], x, s["codesd"], s["alphad"], scale=s["scaled"],
                                                          bias=s["biasd"])
        return tbn.conv2d_fwd(s["desc2"], a, s["codes2"], s["alpha2"], scale=s["scale2"], bias=s["bias2"], residual=sc,
                              relu=True)
    if kind == "fc":
        return tbn.conv2d_fwd(s["desc"], s["x"], s["codes"], s["alpha"], bias=s["bias"])
    if kind == "i8":
        q = tbn.quantize_act_i8(s["x"], 1.0 / s["scale"])
        return {"q": q, "y": tbn.conv2d_fwd_i8(s["desc"], q, s["codes"], s["alpha"], s["scale"], relu=True)}
    if kind == "fp8":
        q = tbn.quantize_act_fp8(s["x"], 1.0 / s["scale"])
        return {"q": q, "y": tbn.conv2d_fwd_fp8(s["desc"], q, s["codes"], s["alpha"], s["scale"], relu=True)}
    return s["net"].forward(s["x"])


# ------------------------------------------------------------------------- the same in 64 bits
def _levels(w):
    """Eq. 3 and 5: the levels in {-2, -1, 1, 2} and the scale of each filter, in fp64."""
    w = w.double()
    q = torch.where(w > 0, 1.0, -1.0).double() * torch.where(w.abs() > 1, 2.0, 1.0).double()
    return q, (w * q).sum(1) / (q * q).sum(1)


def _taps(x, r, stride, pad, p, q):
    xp = F.pad(x, (0, 0, pad, pad, pad, pad))
    for i in range(r):
        for j in range(r):
            yield i, j, xp[:, i:i + (p - 1) * stride + 1:stride, j:j + (q - 1) * stride + 1:stride, :]


def _conv(x, w, r, stride=1, pad=0):
    """NHWC convolution with filters [K][r * r * C], one matrix product a tap."""
    x = x.double()
    n, h, wd, c = x.shape
    p, q = (h + 2 * pad - r) // stride + 1, (wd + 2 * pad - r) // stride + 1
    w = w.double().view(-1, r, r, c)
    y = torch.zeros(n * p * q, w.shape[0], dtype=torch.float64, device=x.device)
    for i, j, t in _taps(x, r, stride, pad, p, q):
        y.addmm_(t.reshape(-1, c), w[:, i, j].t())
    return y.view(n, p, q, -1)


def _conv_back(x, dy, w, r, pad):
    """Gradients of _conv (stride 1) to its input and its filters."""
    x, dy = x.double(), dy.double()
    n, h, wd, c = x.shape
    k = dy.shape[-1]
    p, q = dy.shape[1], dy.shape[2]
    w = w.double().view(k, r, r, c)
    g, dw = dy.reshape(-1, k), torch.zeros(k, r, r, c, dtype=torch.float64, device=x.device)
    dxp = torch.zeros(n, h + 2 * pad, wd + 2 * pad, c, dtype=torch.float64, device=x.device)
    for i, j, t in _taps(x, r, 1, pad, p, q):
        dw[:, i, j] = g.t() @ t.reshape(-1, c)
        dxp[:, i:i + p, j:j + q] += (g @ w[:, i, j]).view(n, p, q, c)
    return dxp[:, pad:pad + h, pad:pad + wd].contiguous(), dw


def _conv2(x, w, r, stride, pad, scale=None, bias=None):
    lv, alpha = _levels(w)
    y = _conv(x, lv * alpha[:, None], r, stride, pad)
    y = y * scale.double() if scale is not None else y
    return y + bias.double() if bias is not None else y


def exact(case, seed):
    t = _inputs(case, seed)
    kind = case["kind"]
    if kind == "first":
        return _conv2(t["x"].to(torch.bfloat16), t["w"], case["r"], case["stride"], case["pad"])
    if kind == "train":
        lv, alpha = _levels(t["w"])
        w = lv * alpha[:, None]
        y = _conv(t["x"], w, case["r"], 1, case["pad"])
        dx, dw = _conv_back(t["x"], t["dy"], w, case["r"], case["pad"])
        v = dw.view(t["w"].shape) + WD * t["w"].double()
        neww = t["w"].double() - LR * v
        if case["fused"]:
            alpha = _levels(neww)[1]
        return {"y": y, "dx": dx if case["c"] >= 8 else None, "dw": dw, "w": neww, "v": v, "codes": None,
                "alpha": alpha}
    if kind == "glue":
        out, x = {}, t["x"].double()
        a, c = x, case["c"]
        if case["bn"]:
            mean, var = x.mean((0, 1, 2)), x.var((0, 1, 2), unbiased=False)
            inv = 1 / torch.sqrt(var + 1e-5)
            xh = (x - mean) * inv
            a = torch.relu(xh * t["gamma"].double() + t["beta"].double())
            out.update(a=a, mean=mean, inv=inv)
            a = a.to(torch.bfloat16).double()  # the tensor that the next call is given
        da = t["dy"].double()
        if case["pool"]:
            k, st, pad = (2, 2, 0) if case["pool"] == 2 else (3, 2, 1)
            h, w = case["h"], case["w"]
            p, q = _pooled(case)
            big = F.pad(a, (0, 0, pad, k, pad, k), value=-math.inf)
            pos = torch.arange(big.shape[1], device=x.device)[:, None] - pad
            pos = pos * w + torch.arange(big.shape[2], device=x.device)[None, :] - pad
            best = torch.full((case["n"], p, q, c), -math.inf, dtype=torch.float64, device=x.device)
            arg = torch.zeros(best.shape, dtype=torch.int64, device=x.device)
            for i in range(k):  # the first of equal values in row-major order
                for j in range(k):
                    v = big[:, i:i + (p - 1) * st + 1:st, j:j + (q - 1) * st + 1:st]
                    at = pos[i:i + (p - 1) * st + 1:st, j:j + (q - 1) * st + 1:st][None, :, :, None].expand_as(arg)
                    new = v > best
                    best, arg = torch.where(new, v, best), torch.where(new, at, arg)
            out["p"], out["arg"] = best, arg.to(torch.int32)
            da = torch.zeros(case["n"], h * w, c, dtype=torch.float64, device=x.device)
            da.scatter_add_(1, arg.view(case["n"], p * q, c), t["dy"].double().view(case["n"], p * q, c))
            da = da.view(x.shape)
            if case["pool"] == 3:
                da = da.to(torch.bfloat16).double()
        if not case["bn"]:
            out["dx"] = torch.where(a > 0, da, torch.zeros_like(da))
            return out
        g = torch.where(a > 0, da, torch.zeros_like(da))
        out["dbeta"], out["dgamma"] = g.sum((0, 1, 2)), (g * xh).sum((0, 1, 2))
        m = x.numel() // c
        out["dx"] = t["gamma"].double() * inv * (g - out["dbeta"] / m - xh * out["dgamma"] / m)
        return out
    if kind == "head":
        n, k, e = case["n"], case["k"], case["h"] ** 2 * case["c"]
        lv, alpha = _levels(t["w"])
        w = lv * alpha[:, None]
        x = t["x"].double().view(n, e)
        z = x @ w.t()
        lse = torch.logsumexp(z, 1)
        lab = t["labels"].long()
        loss = (lse - z.gather(1, lab[:, None])[:, 0]).mean().view(1)
        dz = (torch.exp(z - lse[:, None]) - F.one_hot(lab, k)) / n
        dx = (dz @ w).view(n, case["h"], case["h"], case["c"])
        return {"z": z.view(n, 1, 1, k), "loss": loss, "dz": dz.view(n, 1, 1, k), "dx": dx,
                "dw": (dz.t() @ x).view(k, case["h"], case["h"], case["c"])}
    if kind == "block":
        a = torch.relu(_conv2(t["x"], t["w1"], 3, case["stride"], 1, t["scale1"], t["bias1"]))
        sc = t["x"].double()
        if case["stride"] != 1:
            sc = _conv2(sc, t["wd"], 1, case["stride"], 0, t["scaled"], t["biasd"])
        return torch.relu(_conv2(a, t["w2"], 3, 1, 1, t["scale2"], t["bias2"]) + sc)
    if kind == "fc":
        return _conv2(t["x"], t["w"], 1, 1, 0, None, t["bias"])
    if kind in ("i8", "fp8"):
        f = t["x"].float() * torch.tensor(1.0 / t["scale"], dtype=torch.float32, device="cuda")
        if kind == "i8":
            q = v = torch.round(f).clamp(-127, 127).to(torch.int8)
        else:
            v = f.clamp(-448, 448).to(torch.float8_e4m3fn)
            q, v = v.view(torch.uint8), v.float()
        y = _conv2(v, t["w"], case["r"], 1, case["r"] // 2) * t["scale"]
        return {"q": q, "y": torch.relu(y)}
    layers = {a[0]: a for a in _resnet_layers(case)}

    def conv(name, x):
        _, cin, cout, k, s, p, *_ = layers[name]
        return _conv2(x, t[name][0], k, s, p, t[name][1], t[name][2])

    h = torch.relu(conv("stem", t["x"]))
    h = F.max_pool2d(h.permute(0, 3, 1, 2), 3, 2, 1).permute(0, 2, 3, 1)
    for b in ("layer%d.%d" % (i, j) for i in (1, 2, 3, 4) for j in (0, 1)):
        a = torch.relu(conv(b + ".conv1", h))
        sc = conv(b + ".downsample", h) if b + ".downsample" in layers else h
        h = torch.relu(conv(b + ".conv2", a) + sc)
    return _conv2(h.mean((1, 2))[:, None, None, :], t["fc"][0], 1, 1, 0, None, t["fc"][2]).view(case["n"], 1000)


def tolerance(case):
    """About four times the measured distance of the outputs from exact(): bf16 results are 1.7e-3 off
    (their rounding), gradients to an input 2.4e-3 (the scale's rounding to bf16 too), a network's
    logits 2e-3; one unit in the last place of bf16 is 7.8e-3 of a value.  `differ` is for packed
    words of codes whose weight the update leaves next to a threshold, and for ties of a maximum."""
    return {"rel": 1e-2, "max": 3e-2, "differ": 1e-3}
