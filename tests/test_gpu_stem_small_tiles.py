"""The bf16 stem kernel with the tiles that it takes where they are few (64 pixels, 128 for at most 32 channels) against
the oracle, every output: each instance, tiles that cross images and end past the last one, channels that end inside a
tile, the number of workgroups on both sides of the rule's limit.  Bounds as for every single operator."""
import pytest

import oracle
import tvg_inputs as ti
from _util import check, dev_inputs, to_host

pytestmark = pytest.mark.gpu

# (n, h, w, oc, filter), output channels and pixels per tile; the last five are 520, 504, 520, 448 and 512 tiles of
# 64 pixels (128 for 32 channels) around the limit of 512
SHAPES = [((1, 32, 40, 33, 7), (64, 64)), ((5, 38, 40, 70, 7), (64, 64)), ((2, 112, 112, 64, 7), (64, 64)), ((1, 30, 32, 31, 3), (32, 128)),
          ((5, 34, 40, 17, 3), (32, 128)), ((3, 47, 40, 40, 3), (64, 64)), ((2, 66, 48, 130, 3), (64, 64)), ((10, 128, 104, 64, 7), (64, 256)),
          ((9, 128, 112, 64, 7), (64, 64)), ((20, 128, 104, 32, 3), (32, 256)), ((16, 128, 112, 32, 3), (32, 128)), ((8, 128, 128, 50, 3), (64, 64))]


@pytest.mark.parametrize("tail", ["plain", "bias+residual"])
@pytest.mark.parametrize("cfg,tile", SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_stem_few_tiles(tvg, cfg, tile, tail):
    n, h, w, oc, r = cfg
    full = tail != "plain"
    desc = tvg.ConvDesc(n, 3, h, w, oc, r, r, 2, 2, r // 2, r // 2, tvg.TVG_BF16, 0)
    assert tvg.tvg_conv2d_get_plan(desc) == (3, *tile) and tvg.tvg_conv2d_get_knobs(desc)[:2] == tile
    inp = ti.make_inputs(ti.ConvShape("stem", n, 3, h, w, oc, r, r, 2, r // 2), 9500 + sum(cfg), "bf16", residual=full, bias=full)
    d = dev_inputs(inp, "bf16")
    y = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], d["bias"], d["residual"], stride=2, pad=r // 2, relu=full)
    want = oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"], inp["residual"],
                               stride=(2, 2), pad=(r // 2,) * 2, relu=full)
    check(to_host(y), want, "bf16", cfg)
