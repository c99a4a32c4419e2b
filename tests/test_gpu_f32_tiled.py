"""The fp32 kernel that stages input rows and weight runs in LDS (plan: generic) against the oracle, every
output, at the edges of its tiling: channels that end inside a chunk and a tile, maps that end inside a
pixel tile, one and several chunks, tiles of one row and of many, strides, filters without padding, rows
that fill the patch.  Bounds as for every single operator (tests/_util.py)."""
import pytest

import oracle
import tvg_inputs as ti
from _util import check, dev_inputs, to_host

pytestmark = pytest.mark.gpu

# n, ic, h, w, oc, r, stride, pad
SHAPES = [
    (32, 16, 28, 28, 128, 3, 1, 1), (9, 87, 45, 37, 121, 3, 1, 1), (27, 15, 61, 97, 62, 3, 2, 1),
    (14, 16, 64, 63, 62, 3, 1, 0), (16, 23, 28, 57, 128, 3, 2, 2), (8, 64, 55, 57, 126, 1, 1, 0),
    (16, 60, 57, 31, 128, 1, 2, 0), (7, 95, 65, 64, 128, 1, 1, 0), (16, 8, 63, 41, 125, 5, 1, 2),
    (16, 8, 99, 80, 64, 5, 2, 1), (5, 4, 77, 76, 127, 7, 1, 3), (17, 4, 90, 66, 64, 7, 2, 3),
    (256, 16, 7, 8, 64, 3, 1, 1), (30, 40, 3, 170, 60, 3, 1, 1), (256, 40, 7, 9, 62, 3, 1, 1),
]


@pytest.mark.parametrize("tail", ["plain", "bias+residual"])
@pytest.mark.parametrize("cfg", SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_f32_tiled(tvg, cfg, tail):
    n, ic, h, w, oc, r, stride, pad = cfg
    sh = ti.ConvShape("tiled", n, ic, h, w, oc, r, r, stride, pad)
    desc = tvg.ConvDesc(n, ic, h, w, oc, r, r, stride, stride, pad, pad, tvg.TVG_F32, 0)
    plan = tvg.tvg_conv2d_get_plan(desc)
    assert plan[0] == 0 and plan[1] == 64 and tvg.tvg_conv2d_workspace_size(desc) == 0
    assert not any(tvg.tvg_conv2d_get_knobs(desc))                  # (the gather kernel's are not zero)
    full = tail != "plain"
    inp = ti.make_inputs(sh, 7300 + sum(cfg), "f32", residual=full, bias=full)
    d = dev_inputs(inp, "f32")
    y = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], d["bias"], d["residual"], stride=stride,
                         pad=pad, relu=full)
    want = oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"], inp["residual"],
                               stride=(stride,) * 2, pad=(pad,) * 2, relu=full)
    check(to_host(y), want, "f32", cfg)


# shape and bound on the error against 64 bits (2-norm, relative).  A sum of n random terms one after the other
# has an error of about 2.5e-8 sqrt(n / 2) (2.5e-8: the rms of one fp32 rounding); chains of the kernel's lengths, added up,
# give 6.1e-8, 6.7e-8, 8.8e-8, 1.0e-7 and 1.06e-7 for these, a chunk's products in one chain 9.6e-8 to 2.5e-7.
PRECISION = [((2, 32, 112, 112, 64, 1, 1, 0), 8e-8), ((6, 64, 56, 56, 128, 1, 1, 0), 8.5e-8),
             ((8, 128, 28, 28, 256, 1, 1, 0), 1e-7), ((3, 8, 82, 82, 128, 5, 1, 2), 1.4e-7),
             ((23, 4, 34, 19, 176, 7, 1, 3), 1.5e-7)]


@pytest.mark.parametrize("cfg,bound", PRECISION, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else None)
def test_f32_tiled_sums_in_short_chains(tvg, cfg, bound):
    """The error is that of the kernels which split the reduction over waves, not that of one long sum."""
    import torch
    n, ic, h, w, oc, r, stride, pad = cfg
    desc = tvg.ConvDesc(n, ic, h, w, oc, r, r, stride, stride, pad, pad, tvg.TVG_F32, 0)
    assert tvg.tvg_conv2d_get_plan(desc)[:2] == (0, 64) and not any(tvg.tvg_conv2d_get_knobs(desc))
    inp = ti.make_inputs(ti.ConvShape("sums", n, ic, h, w, oc, r, r, stride, pad), 7400 + sum(cfg), "f32")
    one, none = torch.ones(oc), torch.zeros(oc)
    x, wt = torch.from_numpy(inp["x"]), torch.from_numpy(inp["w"])
    got = tvg.conv2d_fused(x.cuda(), wt.cuda(), one.cuda(), none.cuda(), stride=stride, pad=pad).cpu().double()
    want = torch.nn.functional.conv2d(x.double(), wt.double(), stride=stride, padding=pad)
    err = float((got - want).norm() / want.norm())
    assert err <= bound, (cfg, err)


# (n, ic, h, w, oc, r, stride, pad), pixels per tile: every instance of the kernel - filter, tile, patch size and, for 1x1,
# the three ways of summing a chunk
EVERY_INSTANCE = [
    ((90, 32, 90, 30, 58, 1, 3, 0), 64), ((13, 31, 45, 170, 64, 1, 2, 0), 64), ((32, 64, 3, 64, 128, 1, 1, 0), 64),
    ((8, 72, 31, 28, 121, 1, 1, 0), 64), ((40, 256, 5, 63, 50, 1, 1, 0), 64),
    ((256, 24, 13, 63, 125, 1, 3, 0), 128), ((128, 24, 28, 30, 125, 1, 2, 0), 128),
    ((64, 72, 31, 14, 121, 1, 1, 0), 128), ((128, 256, 1, 77, 256, 1, 1, 0), 128),
    ((256, 8, 5, 45, 64, 3, 3, 2), 64), ((5, 7, 65, 57, 190, 3, 2, 1), 64), ((8, 7, 56, 8, 256, 3, 1, 1), 64),
    ((128, 8, 9, 57, 64, 3, 1, 0), 128), ((128, 7, 56, 4, 126, 3, 1, 1), 128),
    ((128, 8, 28, 77, 50, 3, 2, 0), 128), ((8, 4, 19, 100, 256, 5, 2, 0), 64), ((32, 7, 13, 19, 126, 5, 1, 2), 64),
    ((64, 3, 28, 100, 64, 5, 3, 0), 64), ((256, 3, 63, 8, 128, 5, 2, 2), 128),
    ((128, 4, 14, 14, 126, 5, 1, 2), 128), ((256, 4, 56, 13, 125, 5, 3, 3), 128),
    ((8, 4, 28, 8, 256, 7, 1, 5), 64), ((40, 4, 45, 31, 120, 7, 3, 3), 64), ((5, 7, 28, 112, 256, 7, 2, 2), 64),
    ((256, 4, 14, 4, 128, 7, 1, 4), 128), ((128, 4, 14, 77, 128, 7, 3, 6), 128),
    ((128, 4, 19, 45, 127, 7, 2, 2), 128),
]


@pytest.mark.parametrize("cfg,nt", EVERY_INSTANCE, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_f32_tiled_every_instance(tvg, cfg, nt):
    n, ic, h, w, oc, r, stride, pad = cfg
    desc = tvg.ConvDesc(n, ic, h, w, oc, r, r, stride, stride, pad, pad, tvg.TVG_F32, 0)
    assert tvg.tvg_conv2d_get_plan(desc) == (0, 64, nt) and not any(tvg.tvg_conv2d_get_knobs(desc))
    inp = ti.make_inputs(ti.ConvShape("tiled", n, ic, h, w, oc, r, r, stride, pad), 7500 + sum(cfg), "f32", residual=True, bias=True)
    d = dev_inputs(inp, "f32")
    y = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], d["bias"], d["residual"], stride=stride,
                         pad=pad, relu=True)
    want = oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"], inp["residual"],
                               stride=(stride,) * 2, pad=(pad,) * 2, relu=True)
    check(to_host(y), want, "f32", cfg)
