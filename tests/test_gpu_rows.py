"""The bf16 kernel for problems with few tiles (plan: 3x3 or 1x1 with 16-channel tiles) against the oracle,
every output: each instance (filter, stride, even and odd rows, pixel blocks, loads per lane, waves per
filter row), ragged channels, tiles that end inside an image and tiles over several images.  Bounds as
for every single operator (tests/_util.py)."""
import numpy as np
import pytest

import oracle
import tvg_inputs as ti
from _util import check, dev_inputs, to_dev, to_host

pytestmark = pytest.mark.gpu

# (n, ic, h, w, oc, stride, filter), pixels per tile
EVERY_INSTANCE = [
    ((4, 96, 13, 2, 17, 1, 1), 16), ((3, 96, 1, 22, 33, 1, 1), 32), ((1, 96, 1, 34, 40, 1, 1), 64),
    ((14, 512, 31, 10, 17, 1, 1), 64), ((2, 96, 5, 5, 33, 1, 1), 16), ((1, 96, 1, 27, 33, 1, 1), 32),
    ((1, 96, 1, 43, 17, 1, 1), 64), ((16, 512, 17, 17, 1, 1, 1), 64), ((2, 96, 6, 6, 17, 2, 1), 16),
    ((1, 96, 1, 46, 33, 2, 1), 32), ((16, 256, 34, 34, 1, 2, 1), 64), ((2, 96, 5, 5, 17, 2, 1), 16),
    ((1, 96, 1, 45, 33, 2, 1), 32), ((16, 256, 33, 33, 1, 2, 1), 64), ((2, 96, 15, 2, 17, 1, 3), 16),
    ((4, 32, 6, 4, 17, 1, 3), 16), ((7, 96, 1, 2, 33, 1, 3), 16), ((4, 64, 1, 4, 17, 1, 3), 16),
    ((16, 288, 28, 12, 1, 1, 3), 32), ((1, 64, 1, 20, 33, 1, 3), 32), ((1, 96, 1, 32, 17, 1, 3), 32),
    ((16, 64, 30, 2, 33, 1, 3), 32), ((1, 32, 1, 38, 17, 1, 3), 64), ((1, 96, 1, 34, 17, 1, 3), 64),
    ((16, 64, 23, 20, 1, 1, 3), 64), ((1, 96, 1, 48, 17, 1, 3), 64), ((2, 96, 3, 7, 17, 1, 3), 16),
    ((2, 32, 5, 5, 33, 1, 3), 16), ((3, 96, 1, 1, 17, 1, 3), 16), ((4, 32, 1, 1, 33, 1, 3), 16),
    ((16, 288, 18, 11, 1, 1, 3), 32), ((1, 32, 1, 29, 17, 1, 3), 32), ((1, 96, 1, 23, 33, 1, 3), 32),
    ((16, 64, 29, 3, 33, 1, 3), 32), ((1, 32, 1, 63, 17, 1, 3), 64), ((1, 96, 1, 37, 17, 1, 3), 64),
    ((1, 128, 6, 4, 17, 2, 3), 16), ((2, 32, 6, 4, 33, 2, 3), 16), ((2, 96, 12, 2, 17, 2, 3), 16),
    ((4, 32, 2, 2, 33, 2, 3), 16), ((1, 32, 1, 40, 17, 2, 3), 32), ((1, 96, 1, 38, 17, 2, 3), 32),
    ((16, 64, 21, 22, 17, 2, 3), 32), ((1, 96, 1, 60, 33, 2, 3), 32), ((1, 96, 5, 5, 17, 2, 3), 16),
    ((2, 32, 5, 5, 33, 2, 3), 16), ((2, 96, 4, 5, 17, 2, 3), 16), ((4, 32, 1, 1, 33, 2, 3), 16),
    ((1, 32, 1, 33, 17, 2, 3), 32), ((1, 128, 1, 35, 33, 2, 3), 32), ((16, 64, 21, 21, 17, 2, 3), 32),
    ((1, 96, 1, 47, 17, 2, 3), 32),
    # (twelve loads per lane in tiles of 32 pixels)
    ((33, 576, 1, 1, 579, 1, 3), 32), ((62, 384, 1, 2, 324, 1, 3), 32),
    # reductions longer than a workgroup's waves: several turns per wave
    ((2, 512, 7, 7, 40, 1, 3), 16), ((1, 800, 9, 12, 33, 2, 3), 16), ((3, 1024, 7, 7, 50, 1, 1), 16),
]


@pytest.mark.parametrize("tail", ["plain", "bias+residual"])
@pytest.mark.parametrize("cfg,nt", EVERY_INSTANCE, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_few_tiles_every_instance(tvg, cfg, nt, tail):
    n, ic, h, w, oc, stride, r = cfg
    pad = r // 2
    desc = tvg.ConvDesc(n, ic, h, w, oc, r, r, stride, stride, pad, pad, tvg.TVG_BF16, 0)
    assert tvg.tvg_conv2d_get_plan(desc) == (1 if r == 3 else 4, 16, nt) and not any(tvg.tvg_conv2d_get_knobs(desc))
    full = tail != "plain"
    inp = ti.make_inputs(ti.ConvShape("rows", n, ic, h, w, oc, r, r, stride, pad), 8100 + sum(cfg), "bf16", residual=full, bias=full)
    d = dev_inputs(inp, "bf16")
    y = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], d["bias"], d["residual"], stride=stride, pad=pad, relu=full)
    want = oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"], inp["residual"],
                               stride=(stride,) * 2, pad=(pad,) * 2, relu=full)
    check(to_host(y), want, "bf16", cfg)


@pytest.mark.parametrize("cfg", [(3, 96, 7, 7, 40, 1, 3), (4, 128, 14, 14, 33, 2, 3), (5, 64, 9, 11, 17, 1, 3), (4, 512, 7, 7, 24, 1, 1)],
                         ids=lambda c: "x".join(map(str, c)))
def test_few_tiles_infinities_and_equal_images(tvg, cfg):
    """Equal images of a batch get equal results, wherever their tiles begin; an infinity in the last one
    reaches the outputs whose window holds it and no others."""
    import torch
    n, ic, h, w, oc, stride, r = cfg
    inp = ti.make_inputs(ti.ConvShape("rows", n, ic, h, w, oc, r, r, stride, r // 2), 8300 + sum(cfg), "bf16")
    inp["x"][:] = inp["x"][:1]
    d = dev_inputs(inp, "bf16")
    y = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], stride=stride, pad=r // 2)
    assert torch.equal(y, y[:1].expand_as(y))
    d["x"][n - 1, ic - 1, h - 1, w - 1] = float("inf")
    z = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], stride=stride, pad=r // 2, relu=False)
    clean = tvg.conv2d_fused(d["x"][:1].expand_as(d["x"]).contiguous(), d["w"], d["scale"], d["shift"], stride=stride, pad=r // 2, relu=False)
    hit = torch.zeros(z.shape, dtype=torch.bool)
    for oy in range(z.shape[2]):
        for ox in range(z.shape[3]):
            hit[n - 1, :, oy, ox] = abs(oy * stride - (h - 1)) <= r // 2 and abs(ox * stride - (w - 1)) <= r // 2
    hit = hit.to(z.device)
    assert torch.equal(z[~hit], clean[~hit]) and not bool(torch.isfinite(z[hit]).any())


@pytest.mark.parametrize("cfg", [(1, 64, 56, 56, 128, 128), (2, 128, 28, 28, 256, 256), (3, 256, 14, 14, 128, 40), (2, 96, 13, 11, 64, 70)],
                         ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("centre", [True, False])
def test_few_tiles_two_heads_have_the_bits_of_separate_calls(tvg, cfg, centre):
    import torch
    n, ic, h, w, k1, k2 = cfg
    a = ti.make_inputs(ti.ConvShape("h1", n, ic, h, w, k1, 3, 3, 2, 1), 8500 + sum(cfg), "bf16", residual=True)
    b = ti.make_inputs(ti.ConvShape("h2", n, ic, h, w, k2, 1 if centre else 3, 1 if centre else 3, 2, 0 if centre else 1), 8600 + sum(cfg), "bf16")
    d1, d2 = dev_inputs(a, "bf16"), dev_inputs(b, "bf16")
    w2 = b["w"]
    if centre:
        w2 = np.zeros((k2, ic, 3, 3), np.float32)
        w2[:, :, 1, 1] = b["w"][:, :, 0, 0]
    wt = to_dev(np.concatenate([a["w"], w2]), "bf16")
    scale, shift = torch.cat([d1["scale"], d2["scale"]]), torch.cat([d1["shift"], d2["shift"]])
    want1 = tvg.conv2d_fused(d1["x"], d1["w"], d1["scale"], d1["shift"], None, d1["residual"], stride=2, pad=1, relu=True)
    want2 = tvg.conv2d_fused(d1["x"], d2["w"], d2["scale"], d2["shift"], stride=2, pad=0 if centre else 1, relu=False)
    y1, y2 = torch.empty_like(want1), torch.empty_like(want2)
    desc = tvg.ConvDesc(n, ic, h, w, k1 + k2, 3, 3, 2, 2, 1, 1, tvg.TVG_BF16, tvg.TVG_RELU)
    rc = tvg.tvg_conv2d_fused_dual(desc, k1, tvg.TVG_CENTRE_TAP_ONLY if centre else 0, d1["x"], wt, scale, shift, None, d1["residual"], y1, y2)
    assert rc == 0, tvg.status_string(rc)
    assert torch.equal(y1, want1) and torch.equal(y2, want2)


# ..., which of the two heads runs in the kernel for few tiles when it is called by itself
@pytest.mark.parametrize("cfg,few", [
    ((6, 64, 56, 56, 128, 128, 2), (False, False)), ((12, 256, 14, 14, 512, 512, 2), (False, False)), ((8, 160, 14, 14, 512, 512, 2), (False, True)),
    ((4, 64, 28, 28, 64, 2048, 2), (True, False)), ((1, 256, 112, 112, 64, 16, 1), (False, True)), ((2, 96, 13, 11, 64, 70, 1), (True, True)),
    ((3, 512, 14, 14, 64, 40, 1), (True, True)), ((5, 160, 8, 127, 64, 24, 2), (False, True)), ((5, 160, 8, 128, 64, 17, 2), (False, True)),
    # both in one launch: the other instances (one or two blocks of pixels, loads per lane, even and odd rows, filter rows)
    ((1, 256, 2, 12, 64, 1, 2), (True, True)), ((16, 64, 1, 8, 64, 1, 2), (True, True)), ((3, 512, 11, 36, 128, 64, 2), (True, True)),
    ((16, 64, 16, 24, 64, 1, 2), (True, True)), ((2, 192, 2, 5, 256, 1, 2), (True, True)), ((18, 32, 14, 5, 64, 17, 2), (True, True)),
    ((54, 32, 2, 3, 128, 128, 2), (True, True)), ((3, 256, 27, 15, 256, 128, 2), (True, True)), ((5, 32, 26, 35, 64, 17, 2), (True, False)),
    ((2, 512, 13, 35, 256, 17, 2), (True, True)), ((3, 64, 18, 29, 256, 1, 2), (True, True)),
    ((2, 64, 28, 28, 64, 1024, 2), (True, True)), ((1, 64, 28, 28, 64, 40, 1), (True, False)), ((2, 128, 28, 28, 192, 70, 1), (True, False)), ((8, 128, 28, 28, 192, 70, 1), (False, False)), ((4, 128, 28, 28, 256, 256, 2), (True, True)), ((32, 64, 56, 56, 128, 128, 2), (False, False)),
], ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("centre", [True, False])
def test_two_heads_have_the_bits_of_separate_calls_whichever_is_split(tvg, cfg, few, centre):
    import torch
    n, ic, h, w, k1, k2, stride = cfg
    r2 = 1 if centre else 3
    g = torch.Generator(device="cuda").manual_seed(8700 + sum(cfg))
    def rand(*shape):
        return torch.rand(shape, generator=g, device="cuda") * 2 - 1
    x, w1, w2 = (rand(*s).to(torch.bfloat16) for s in ((n, ic, h, w), (k1, ic, 3, 3), (k2, ic, r2, r2)))
    scale, shift, bias = rand(k1 + k2), rand(k1 + k2), rand(k1 + k2)
    joined = torch.zeros(k1 + k2, ic, 3, 3, dtype=torch.bfloat16, device="cuda")
    joined[:k1] = w1
    if centre:
        joined[k1:, :, 1, 1] = w2[:, :, 0, 0]
    else:
        joined[k1:] = w2
    if centre:
        d1 = tvg.ConvDesc(n, ic, h, w, k1, 3, 3, stride, stride, 1, 1, tvg.TVG_BF16, 0)
        d2 = tvg.ConvDesc(n, ic, h, w, k2, 1, 1, stride, stride, 0, 0, tvg.TVG_BF16, 0)
        assert (tvg.tvg_conv2d_get_plan(d1)[1] == 16, tvg.tvg_conv2d_get_plan(d2)[1] == 16) == few
    want1 = tvg.conv2d_fused(x, w1, scale[:k1], shift[:k1], bias[:k1], stride=stride, pad=1, relu=True)
    residual = rand(*want1.shape).to(torch.bfloat16)
    want1 = tvg.conv2d_fused(x, w1, scale[:k1], shift[:k1], bias[:k1], residual, stride=stride, pad=1, relu=True)
    want2 = tvg.conv2d_fused(x, w2, scale[k1:].clone(), shift[k1:].clone(), bias[k1:].clone(), stride=stride, pad=r2 // 2, relu=False)
    y1, y2 = torch.full_like(want1, float("nan")), torch.full_like(want2, float("nan"))
    desc = tvg.ConvDesc(n, ic, h, w, k1 + k2, 3, 3, stride, stride, 1, 1, tvg.TVG_BF16, tvg.TVG_RELU)
    rc = tvg.tvg_conv2d_fused_dual(desc, k1, tvg.TVG_CENTRE_TAP_ONLY if centre else 0, x, joined, scale, shift, bias, residual, y1, y2)
    assert rc == 0, tvg.status_string(rc)
    assert torch.equal(y1, want1) and torch.equal(y2, want2)


@pytest.mark.parametrize("dtype,cfg", [("bf16", (2, 128, 28, 28, 128, 1, 3)), ("bf16", (2, 96, 13, 11, 33, 1, 1)), ("bf16", (8, 512, 14, 14, 512, 1, 1)),
                                       ("f32", (1, 512, 14, 14, 512, 1, 1)), ("f32", (8, 256, 28, 28, 256, 1, 1))],
                         ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else c)
def test_store_hint_changes_no_bits(tvg, dtype, cfg):
    import torch
    n, ic, h, w, oc, stride, r = cfg
    d = dev_inputs(ti.make_inputs(ti.ConvShape("hint", n, ic, h, w, oc, r, r, stride, r // 2), 8800 + sum(cfg), dtype, residual=True), dtype)
    for relu in (True, False):
        y, z = (tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], None, d["residual"], stride=stride, pad=r // 2, relu=relu, stream_out=hint)
                for hint in (True, False))
        assert torch.equal(y, z)
        if not relu:
            assert bool((y < 0).any())


@pytest.mark.parametrize("cfg", [(8, 160, 14, 14, 512, 64, 2), (2, 96, 13, 11, 64, 70, 1)], ids=lambda c: "x".join(map(str, c)))
def test_two_heads_of_a_launch_each_in_a_graph(tvg, cfg):
    """Captured once, replayed with other inputs and eager work between: the bits of an eager call every time."""
    import torch
    n, ic, h, w, k1, k2, stride = cfg
    g = torch.Generator(device="cuda").manual_seed(8900 + sum(cfg))
    def rand(*shape):
        return torch.rand(shape, generator=g, device="cuda") * 2 - 1
    x, joined = rand(n, ic, h, w).bfloat16(), torch.zeros(k1 + k2, ic, 3, 3, dtype=torch.bfloat16, device="cuda")
    joined[:k1], joined[k1:, :, 1, 1] = rand(k1, ic, 3, 3).bfloat16(), rand(k2, ic).bfloat16()
    scale, shift = rand(k1 + k2), rand(k1 + k2)
    oh, ow = (h - 1) // stride + 1, (w - 1) // stride + 1
    out = [torch.empty(n, k, oh, ow, dtype=torch.bfloat16, device="cuda") for k in (k1, k2, k1, k2)]
    desc = tvg.ConvDesc(n, ic, h, w, k1 + k2, 3, 3, stride, stride, 1, 1, tvg.TVG_BF16, tvg.TVG_RELU)
    def call(y1, y2):
        assert tvg.tvg_conv2d_fused_dual(desc, k1, tvg.TVG_CENTRE_TAP_ONLY, x, joined, scale, shift, None, None, y1, y2) == 0
    call(*out[2:])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        call(*out[:2])
    for _ in range(3):
        x.copy_(rand(n, ic, h, w))
        call(*out[2:])
        out[0].zero_(), out[1].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[0], out[2]) and torch.equal(out[1], out[3])
