"""The bf16 kernel for any filter, stride, padding and channel count (plan: generic) against the
oracle, every output, at the edges of its tiling: rows narrower than a load and one pixel longer,
maps that end inside a tile and tiles that cross images, one and several channel chunks, a chunk's
surplus units, filters with more taps than the stride and fewer, reductions split over workgroups.
Bounds as for every single operator (tests/_util.py)."""
import pytest

import oracle
import tvg_inputs as ti
from _util import check, dev_inputs, to_host

pytestmark = pytest.mark.gpu

# n, ic, h, w, oc, r, s, stride, pad
SHAPES = [
    (6, 83, 45, 37, 139, 3, 3, 1, 1), (1, 1, 1, 1, 1, 1, 1, 1, 0), (3, 7, 3, 3, 33, 3, 3, 1, 1),
    (3, 9, 6, 4, 31, 3, 3, 1, 1), (2, 17, 5, 9, 65, 5, 5, 1, 2), (9, 33, 7, 7, 64, 3, 3, 1, 1),
    (1, 40, 64, 65, 96, 3, 5, 1, 1), (2, 20, 33, 30, 97, 1, 1, 2, 0), (4, 5, 20, 18, 40, 2, 3, 3, 1),
    (2, 3, 40, 41, 24, 7, 7, 2, 3), (1, 8, 30, 130, 20, 11, 11, 1, 5), (1, 130, 6, 6, 200, 5, 5, 1, 2),
    (2, 300, 9, 9, 40, 7, 7, 1, 3), (1, 9, 20, 20, 16, 15, 16, 1, 7), (40, 24, 3, 5, 70, 3, 3, 2, 0),
]


@pytest.mark.parametrize("tail", ["plain", "bias+residual"])
@pytest.mark.parametrize("cfg", SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_bf16_any_shape(tvg, cfg, tail):
    n, ic, h, w, oc, r, s, stride, pad = cfg
    sh = ti.ConvShape("any", n, ic, h, w, oc, r, s, stride, pad)
    desc = tvg.ConvDesc(n, ic, h, w, oc, r, s, stride, stride, pad, pad, tvg.TVG_BF16, 0)
    assert tvg.tvg_conv2d_get_plan(desc)[0] == 0 and tvg.tvg_conv2d_workspace_size(desc) > 0
    assert not any(tvg.tvg_conv2d_get_knobs(desc))                  # (the gather kernel's are not zero)
    full = tail != "plain"
    inp = ti.make_inputs(sh, 6100 + sum(cfg), "bf16", residual=full, bias=full)
    d = dev_inputs(inp, "bf16")
    y = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], d["bias"], d["residual"], stride=stride,
                         pad=pad, relu=full)
    want = oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"], inp["residual"],
                               stride=(stride,) * 2, pad=(pad,) * 2, relu=full)
    check(to_host(y), want, "bf16", cfg)


# one shape per tile of the kernel, each with units that no tap fills in the last turn of a chunk
WITH_SURPLUS_UNITS = [
    (3, 7, 3, 3, 33, 3, 1, 1), (8, 45, 65, 63, 60, 3, 1, 1), (16, 20, 65, 63, 50, 3, 1, 1),
    (20, 20, 65, 63, 31, 3, 1, 1), (8, 20, 65, 63, 31, 3, 1, 1), (2, 300, 13, 13, 31, 5, 1, 2),
]


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("cfg", WITH_SURPLUS_UNITS, ids=lambda c: "x".join(map(str, c)))
def test_an_infinity_in_x_reaches_its_outputs_and_no_others(tvg, cfg, relu):
    """An overflowed activation: every output whose window holds it is an infinity of the right sign (or 0
    behind the ReLU), every other one is what it is without it.  Reference: torch in 64 bits on the CPU."""
    import torch
    n, ic, h, w, oc, r, stride, pad = cfg
    inp = ti.make_inputs(ti.ConvShape("inf", n, ic, h, w, oc, r, r, stride, pad), 6400 + sum(cfg), "bf16")
    inp["x"][0, 0, 1, 1] = float("inf")
    inp["x"][n - 1, ic - 1, h - 1, w - 1] = float("-inf")
    d = dev_inputs(inp, "bf16")
    got = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], stride=stride, pad=pad, relu=relu).cpu().double()
    t = {k: torch.from_numpy(inp[k]).double() for k in ("x", "w", "scale", "shift")}
    want = torch.nn.functional.conv2d(t["x"], t["w"], stride=stride, padding=pad)
    want = want * t["scale"].view(1, -1, 1, 1) + t["shift"].view(1, -1, 1, 1)
    want = want.relu() if relu else want
    assert bool(torch.isposinf(want).any()) and not bool(torch.isnan(want).any())
    odd = torch.isinf(want)
    assert torch.equal(got[odd], want[odd]) and bool(torch.isfinite(got[~odd]).all())
    check(got[~odd].numpy(), want[~odd].numpy(), "bf16", cfg)


# several chunks of channels; pixel tiles within an image, tiles that cross images, a split reduction
SEVERAL_CHUNKS = [(12, 100, 45, 37, 40, 5, 1, 2), (24, 300, 9, 9, 70, 5, 1, 2), (9, 300, 13, 13, 31, 5, 1, 2),
                  (4, 509, 14, 14, 100, 1, 1, 0)]


@pytest.mark.parametrize("cfg", SEVERAL_CHUNKS, ids=lambda c: "x".join(map(str, c)))
def test_equal_images_of_a_batch_get_equal_results(tvg, cfg):
    """Bit for bit, wherever in the batch (and so in which tile) an image lies."""
    import torch
    n, ic, h, w, oc, r, stride, pad = cfg
    inp = ti.make_inputs(ti.ConvShape("same", n, ic, h, w, oc, r, r, stride, pad), 6700 + sum(cfg), "bf16")
    inp["x"][:] = inp["x"][:1]
    d = dev_inputs(inp, "bf16")
    y = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], stride=stride, pad=pad)
    assert torch.equal(y, y[:1].expand_as(y))


# (n, ic, h, w, oc, r, s, stride, pad), tile: every instance of the kernel - 1, 4 or 8 pixels per load, one or two
# loads per thread under each tile -, tiles within an image and across images, several chunks, a split reduction
EVERY_INSTANCE = [
    ((1, 5, 3, 1, 1, 3, 1, 3, 0), (32, 128)), ((2, 35, 31, 3, 1, 1, 1, 3, 0), (32, 128)),
    ((1, 9, 5, 4, 96, 1, 1, 2, 0), (32, 128)), ((40, 9, 3, 7, 1, 2, 1, 3, 0), (32, 128)),
    ((8, 500, 5, 33, 1, 2, 2, 1, 0), (32, 128)), ((3, 5, 65, 9, 1, 5, 1, 3, 0), (32, 128)),
    ((400, 3, 63, 2, 96, 1, 1, 1, 0), (32, 256)), ((400, 3, 65, 3, 16, 1, 1, 1, 0), (32, 256)),
    ((200, 3, 63, 7, 1, 1, 1, 1, 0), (32, 256)), ((400, 60, 19, 5, 96, 1, 1, 1, 0), (32, 256)),
    ((90, 3, 63, 130, 1, 1, 1, 3, 0), (32, 256)), ((90, 20, 31, 100, 1, 3, 1, 2, 0), (32, 256)),
    ((8, 60, 90, 45, 65, 2, 1, 1, 0), (32, 256)), ((1, 3, 5, 2, 50, 1, 1, 3, 0), (64, 64)),
    ((1, 20, 45, 3, 33, 3, 1, 3, 0), (64, 64)), ((1, 5, 1, 7, 97, 1, 1, 2, 0), (64, 64)),
    ((1, 500, 13, 7, 130, 5, 1, 1, 0), (64, 64)), ((1, 3, 3, 13, 60, 1, 1, 3, 0), (64, 64)),
    ((1, 17, 19, 45, 33, 3, 1, 3, 0), (64, 64)), ((200, 3, 63, 2, 120, 1, 1, 1, 0), (64, 128)),
    ((400, 9, 90, 3, 33, 1, 1, 2, 0), (64, 128)), ((90, 5, 90, 6, 33, 1, 1, 1, 0), (64, 128)),
    ((200, 35, 63, 4, 130, 2, 2, 2, 0), (64, 128)), ((90, 3, 7, 65, 33, 1, 1, 1, 0), (64, 128)),
    ((20, 9, 90, 100, 130, 3, 1, 3, 0), (64, 128)), ((90, 3, 90, 2, 97, 3, 3, 1, 2), (64, 256)),
    ((200, 9, 45, 2, 130, 2, 2, 1, 1), (64, 256)), ((90, 3, 63, 6, 97, 1, 1, 1, 0), (64, 256)),
    ((400, 9, 90, 5, 130, 2, 1, 3, 0), (64, 256)), ((400, 3, 19, 11, 33, 1, 1, 1, 0), (64, 256)),
    ((90, 17, 31, 100, 60, 3, 1, 2, 0), (64, 256)),
]


@pytest.mark.parametrize("cfg,tile", EVERY_INSTANCE, ids=lambda c: "x".join(map(str, c)))
def test_bf16_any_shape_every_instance(tvg, cfg, tile):
    n, ic, h, w, oc, r, s, stride, pad = cfg
    desc = tvg.ConvDesc(n, ic, h, w, oc, r, s, stride, stride, pad, pad, tvg.TVG_BF16, 0)
    assert tvg.tvg_conv2d_get_plan(desc) == (0, *tile) and not any(tvg.tvg_conv2d_get_knobs(desc))
    inp = ti.make_inputs(ti.ConvShape("any", n, ic, h, w, oc, r, s, stride, pad), 6800 + sum(cfg), "bf16", residual=True, bias=True)
    d = dev_inputs(inp, "bf16")
    y = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], d["bias"], d["residual"], stride=stride,
                         pad=pad, relu=True)
    want = oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"], inp["residual"],
                               stride=(stride,) * 2, pad=(pad,) * 2, relu=True)
    check(to_host(y), want, "bf16", cfg)
