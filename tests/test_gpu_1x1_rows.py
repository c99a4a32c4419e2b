"""The bf16 1x1 kernel that stages pixels as they lie in memory (row_loads = 2) against the oracle, every output:
each tile and chunk size, maps of 8n, 4n, 2n and an odd number of pixels, channels that end inside a tile, reductions
shorter than what is in flight, tiles that cross images; unaligned outputs.  Bounds as for every single operator."""
import pytest

import oracle
import tvg_inputs as ti
from _util import check, dev_inputs, to_dev, to_host

pytestmark = pytest.mark.gpu

# n, ic, h, w, oc
SHAPES = [(3, 32, 8, 8, 64), (5, 64, 7, 7, 40), (4, 96, 14, 14, 130), (9, 160, 6, 5, 33), (2, 128, 9, 11, 128),
          (7, 1024, 7, 7, 96), (3, 1088, 4, 9, 65), (1, 256, 1, 1, 17), (33, 32, 3, 1, 64), (2, 320, 13, 26, 200)]


@pytest.mark.parametrize("tail", ["plain", "bias+residual"])
@pytest.mark.parametrize("tile", [(64, 64), (64, 128), (128, 128)], ids=lambda t: "%dx%d" % t)
@pytest.mark.parametrize("cfg", SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_1x1_rows_every_tile(tvg, cfg, tile, tail):
    import torch
    n, ic, h, w, oc = cfg
    oc += 64 if tile[0] == 128 else 0                   # (128-channel tiles from 65 channels on)
    full = tail != "plain"
    desc = tvg.ConvDesc(n, ic, h, w, oc, 1, 1, 1, 1, 0, 0, tvg.TVG_BF16, tvg.TVG_RELU if full else 0)
    inp = ti.make_inputs(ti.ConvShape("pwr", n, ic, h, w, oc, 1, 1, 1, 0), 9100 + sum(cfg), "bf16", residual=full, bias=full)
    d = dev_inputs(inp, "bf16")
    want = oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"], inp["residual"],
                               stride=(1, 1), pad=(0, 0), relu=full)
    assert tvg.tvg_conv2d_set_knobs(desc, (*tile, 1, 0, 0, 2)) == 0
    try:
        assert tvg.tvg_conv2d_get_plan(desc) == (4, *tile) and tvg.tvg_conv2d_get_knobs(desc) == (*tile, 1, 0, 0, 2)
        for off in (0, 1):                              # y and the residual at an even and at an odd element
            def at(t):
                store = torch.zeros(t.numel() + 8, dtype=torch.bfloat16, device="cuda")
                v = store[off:off + t.numel()].view(t.shape)
                v.copy_(t)
                return v
            y = at(torch.zeros((n, oc, h, w), dtype=torch.bfloat16, device="cuda"))
            rc = tvg.tvg_conv2d_fused(desc, d["x"], d["w"], d["scale"], d["shift"], d["bias"], at(d["residual"]) if full else None, y, None, 0, None)
            assert rc == 0, tvg.status_string(rc)
            check(to_host(y), want, "bf16", (cfg, tile, off))
    finally:
        tvg.tvg_conv2d_set_knobs(desc, None)


@pytest.mark.parametrize("kw,plan", [(dict(n=32, c=512, h=14, w=14, k=512), (4, 64, 128)), (dict(n=32, c=1024, h=7, w=7, k=1024), (4, 64, 64)),
                                     (dict(n=128, c=1024, h=7, w=7, k=1024), (4, 128, 128)), (dict(n=32, c=32, h=112, w=112, k=64), (4, 64, 128))])
def test_1x1_rows_plans(tvg, kw, plan):
    """What the rule takes, and that the reported knobs, fixed, change nothing; a tile alone is the other kernel's."""
    desc = tvg.ConvDesc(kw["n"], kw["c"], kw["h"], kw["w"], kw["k"], 1, 1, 1, 1, 0, 0, tvg.TVG_BF16, 0)
    knobs = tvg.tvg_conv2d_get_knobs(desc)
    assert tvg.tvg_conv2d_get_plan(desc) == plan and knobs == (plan[1], plan[2], 1, 0, 0, 2)
    try:
        assert tvg.tvg_conv2d_set_knobs(desc, knobs) == 0
        assert tvg.tvg_conv2d_get_plan(desc) == plan and tvg.tvg_conv2d_get_knobs(desc) == knobs
        assert tvg.tvg_conv2d_set_knobs(desc, None) == 0 and tvg.tvg_conv2d_set_tile(desc, 64, 64) == 0
        assert tvg.tvg_conv2d_get_knobs(desc) == (64, 64, 1, 0, 0, 0)
    finally:
        tvg.tvg_conv2d_set_knobs(desc, None)


def test_1x1_rows_infinity_stays_in_its_pixel(tvg):
    import torch
    inp = ti.make_inputs(ti.ConvShape("pwr", 3, 256, 14, 14, 128, 1, 1, 1, 0), 9300, "bf16")
    d = dev_inputs(inp, "bf16")
    clean = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], relu=False)
    d["x"][1, 3, 13, 13] = float("inf")
    y = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], relu=False)
    assert not bool(torch.isfinite(y[1, :, 13, 13]).any())
    y[1, :, 13, 13] = clean[1, :, 13, 13]
    assert torch.equal(y, clean)
