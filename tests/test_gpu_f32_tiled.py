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
    (32, 16, 28, 28, 128, 3, 1, 1), (9, 87, 45, 37, 121, 3, 1, 1), (24, 15, 61, 97, 60, 3, 2, 1),
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
    full = tail != "plain"
    inp = ti.make_inputs(sh, 7300 + sum(cfg), "f32", residual=full, bias=full)
    d = dev_inputs(inp, "f32")
    y = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], d["bias"], d["residual"], stride=stride,
                         pad=pad, relu=full)
    want = oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"], inp["residual"],
                               stride=(stride,) * 2, pad=(pad,) * 2, relu=full)
    check(to_host(y), want, "f32", cfg)
