"""The stem with its pooling in one pass: bit for bit the two separate passes (the same sums in the same
order, a maximum of the same bf16 values), over kernel sizes, strides, borders, odd and even output sizes
against the 8 x 30 tiles, one and several tiles each way, channel paddings, filters past one block,
segments that begin below the top, and inputs that overflow.  Layers without a fused form are refused."""
import pytest
import torch

from test_gpu_parity import log

pytestmark = pytest.mark.gpu

CASES = [
    # n, h, w, c, k, r, stride, pad
    (8, 224, 224, 3, 64, 7, 2, 3),
    (25, 119, 121, 3, 64, 7, 2, 3),
    (1, 1000, 400, 3, 64, 7, 2, 3),       # few columns of tiles: many segments
    (300, 32, 37, 3, 24, 5, 1, 2),
    (600, 61, 31, 2, 72, 7, 2, 3),        # two blocks of filters
    (3, 420, 421, 2, 56, 5, 2, 0),
    (2100, 13, 13, 3, 64, 3, 1, 1),
    (40, 70, 75, 5, 40, 3, 1, 1),
    (3, 500, 800, 3, 136, 3, 1, 1),
    (4200, 9, 10, 3, 64, 7, 2, 3),        # less than one tile
]


@pytest.mark.parametrize("epilogue", [True, False])
@pytest.mark.parametrize("geom", CASES, ids=str)
def test_stem_pool_equals_the_two_passes(tbn, geom, epilogue):
    log("stem with pooling %s" % (geom,))
    n, h, w, c, k, r, st, pd = geom
    desc = tbn.ConvDesc(*geom[:5], r, r, st, pd)
    g = torch.Generator(device="cuda").manual_seed(sum(geom))
    codes, alpha, _ = tbn.quantize(torch.randn(k, r * r * c, generator=g, device="cuda"))
    kw = {}
    if epilogue:
        kw = dict(scale=torch.rand(k, generator=g, device="cuda") - 0.3, bias=torch.randn(k, generator=g, device="cuda"))
    for dtype in (torch.bfloat16, torch.float32):
        x = torch.randn(n, h, w, c, generator=g, device="cuda")
        x[0, h // 2, w // 2, 0] = float("inf")
        x[-1, 0, -1, 0] = float("nan")
        x = x.to(dtype)
        y = tbn.conv2d_relu_maxpool_fwd(desc, x, codes, alpha, **kw)
        ws = torch.empty(tbn.workspace_size(tbn.OP_FWD, desc), dtype=torch.uint8, device="cuda")
        a = tbn.conv2d_fwd(desc, x, codes, alpha, relu=True, ws=ws, **kw)
        ref, _ = tbn.maxpool2d_fwd(a, 3, 2, 1)
        assert y is not None and y.shape == ref.shape
        assert torch.equal(y.view(torch.int16), ref.view(torch.int16))


@pytest.mark.parametrize("geom", [(1, 224, 224, 3, 64, 7, 2, 3), (8, 224, 224, 3, 60, 7, 2, 3),
                                  (8, 224, 224, 8, 64, 7, 2, 3), (30, 200, 200, 1, 64, 3, 1, 1)], ids=str)
def test_layers_without_a_fused_form(tbn, geom):
    n, h, w, c, k, r, st, pd = geom
    desc = tbn.ConvDesc(*geom[:5], r, r, st, pd)
    x = torch.zeros(n, h, w, c, device="cuda", dtype=torch.bfloat16)
    codes, alpha, _ = tbn.quantize(torch.ones(k, r * r * c, device="cuda"))
    assert tbn.conv2d_relu_maxpool_fwd(desc, x, codes, alpha) is None


def test_network_with_and_without_the_fused_stem(tbn):
    """Captured as a graph too: replays on new inputs, with eager work between them."""
    from paper_1701_00485_amd.networks import ResNet18
    net = ResNet18()
    x = torch.randn(8, 224, 224, 3, device="cuda").bfloat16()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        net.forward(x)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = net.forward(x)
    for i in range(3):
        x.copy_(torch.randn(8, 224, 224, 3, device="cuda").bfloat16())
        graph.replay()
        torch.cuda.synchronize()
        ref = net.forward(x, trace=[])
        assert torch.equal(net.forward(x), ref) and torch.equal(out, ref)
