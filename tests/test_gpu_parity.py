"""GPU parity: the HIP path (through the C ABI) against the fp64 CPU oracle on the same
seeded inputs.  Tolerances: max relative error (see tests/_util.rel_err) 1e-4 for fp32
inputs, 2e-2 for bf16 inputs; bit-exact where the arithmetic is exact."""
import numpy as np
import pytest

import oracle
import tvg_inputs as ti
from _util import BLOCK_TIGHT, TOL, check, dev_inputs, fixed_tile, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


def run_dense(tvg, sh, inp, dtype, relu=True, stream_out=False, tile=""):
    import torch
    d = dev_inputs(inp, dtype)
    with fixed_tile(tvg, sh, dtype, tile):
        y = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], d["bias"], d["residual"],
                             stride=sh.stride, pad=sh.pad, relu=relu, stream_out=stream_out)
        torch.cuda.synchronize()
    return y


def oracle_dense(sh, inp, relu=True, idx=None):
    kw = dict(stride=(sh.stride, sh.stride), pad=(sh.pad, sh.pad), relu=relu)
    if idx is None:
        return oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"],
                                   inp["residual"], **kw)
    return oracle.conv2d_fused_at(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"],
                                  inp["residual"], idx=idx, **kw)


# ------------------------------------------------------------------------------------------
# depthwise (configuration 3: D1..D9, fp32, batch 1)
# ------------------------------------------------------------------------------------------

@pytest.mark.parametrize("i", range(9))
def test_config3_depthwise_fp32_batch1(tvg, i):
    import torch
    sh = ti.mobilenet_depthwise(1)[i]
    inp = ti.make_inputs(sh, ti.layer_seed(3, i), "f32")
    d = dev_inputs(inp, "f32")
    y = tvg.dwconv2d_fused(d["x"], d["w"], d["scale"], d["shift"], stride=sh.stride, pad=1, relu=True)
    hinted = tvg.dwconv2d_fused(d["x"], d["w"], d["scale"], d["shift"], stride=sh.stride, pad=1,
                                relu=True, stream_out=True)
    torch.cuda.synchronize()
    assert torch.equal(y, hinted)                 # the store hint changes no value
    want = oracle.dwconv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"],
                                 stride=(sh.stride,) * 2, pad=(1, 1), relu=True)
    assert tuple(y.shape) == sh.y_shape()
    check(to_host(y), want, "f32")


@pytest.mark.parametrize("i", range(9))
def test_depthwise_bf16_table2_shapes_batch2(tvg, i):
    """D1..D9 in bf16 with residual (the register-blocked bf16 kernel with 8 and 4 columns per
    lane, the small-plane kernel), hinted and plain stores bit-identical."""
    import torch
    sh = ti.mobilenet_depthwise(2)[i]
    inp = ti.make_inputs(sh, ti.layer_seed(3, 200 + i), "bf16", residual=True)
    d = dev_inputs(inp, "bf16")
    y = tvg.dwconv2d_fused(d["x"], d["w"], d["scale"], d["shift"], None, d["residual"],
                           stride=sh.stride, pad=1, relu=True)
    hinted = tvg.dwconv2d_fused(d["x"], d["w"], d["scale"], d["shift"], None, d["residual"],
                                stride=sh.stride, pad=1, relu=True, stream_out=True)
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), hinted.view(torch.int16))
    want = oracle.dwconv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], None,
                                 inp["residual"], stride=(sh.stride,) * 2, pad=(1, 1), relu=True)
    check(to_host(y), want, "bf16")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,c,h,w,stride", [(3, 5, 9, 11, 1), (2, 7, 10, 13, 2), (1, 3, 1, 1, 1),
                                              (2, 70, 33, 65, 2), (1, 2, 130, 131, 1),
                                              (4, 300, 7, 7, 1), (1, 1, 2, 3, 2),
                                              # rows that are multiples of four (fp32: the
                                              # register-blocked kernel), ragged row blocks
                                              (2, 5, 12, 16, 1), (3, 7, 16, 24, 2), (1, 3, 8, 8, 1),
                                              (2, 4, 21, 32, 2), (1, 2, 9, 12, 1), (1, 3, 7, 8, 2),
                                              (2, 6, 30, 120, 1),
                                              # enough lanes for the fp32 kernel's blocks of 2 and 4
                                              # rows, with a ragged last block, and stride 2
                                              (16, 512, 27, 28, 1), (8, 256, 30, 56, 1), (8, 256, 30, 56, 2)])
def test_depthwise_ragged_shapes_full_tail(tvg, dtype, n, c, h, w, stride):
    import torch
    sh = ti.ConvShape("dw", n, c, h, w, c, 3, 3, stride, 1, depthwise=True)
    inp = ti.make_inputs(sh, 4242 + h * w + c, dtype, residual=True, bias=True)
    d = dev_inputs(inp, dtype)
    y = tvg.dwconv2d_fused(d["x"], d["w"], d["scale"], d["shift"], d["bias"], d["residual"],
                           stride=stride, pad=1, relu=True)
    torch.cuda.synchronize()
    want = oracle.dwconv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"],
                                 inp["residual"], stride=(stride,) * 2, pad=(1, 1), relu=True)
    check(to_host(y), want, dtype)


# (n, c, h, w, stride): narrow output rows (14 or 7 pixels) on enough planes for the kernel that
# gives a lane one output row - square and oblong maps, an odd height under stride 2
ROWS_SHAPES = [(8, 256, 14, 14, 1), (4, 512, 9, 14, 1), (8, 300, 7, 7, 1), (8, 256, 28, 28, 2),
               (8, 256, 20, 28, 2), (8, 320, 14, 14, 2), (8, 400, 13, 14, 2), (3, 800, 7, 7, 1),
               (4, 200, 28, 28, 1), (3, 256, 25, 28, 1),      # 28-pixel rows: this kernel in bf16 only
               (3, 801, 7, 7, 1)]      # bf16: 14-byte rows, and a tensor that ends in half a word


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("variant", ["plain", "bias+residual", "no-relu+residual", "offset"])
@pytest.mark.parametrize("cfg", ROWS_SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_depthwise_row_per_lane_kernel_shapes(tvg, cfg, variant, dtype):
    """Every output of the row-per-lane depthwise kernel; "offset" places x, y and the residual
    4 bytes (and, for bf16, also 2 bytes: the fallback) past a 16-byte boundary."""
    import torch
    n, c, h, w, stride = cfg
    sh = ti.ConvShape("dw", n, c, h, w, c, 3, 3, stride, 1, depthwise=True)
    res = variant != "plain"
    inp = ti.make_inputs(sh, 5100 + sum(cfg) + len(variant), dtype, residual=res, bias="bias" in variant)
    relu = "no-relu" not in variant
    want = oracle.dwconv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"],
                                 inp["residual"], stride=(stride,) * 2, pad=(1, 1), relu=relu)
    d = dev_inputs(inp, dtype)
    shifts = [0] if variant != "offset" else ([1] if dtype == "f32" else [2, 1])
    for off in shifts:
        def place(t):
            base = torch.empty(t.numel() + 16, dtype=t.dtype, device=t.device)
            v = base[off:off + t.numel()].view(t.shape)
            v.copy_(t)
            return v
        x, r = (place(d["x"]), place(d["residual"])) if off else (d["x"], d["residual"])
        y = torch.full(sh.y_shape(), float("nan"), dtype=x.dtype, device=x.device)
        y = place(y) if off else y
        for hint in (False, True):
            y.fill_(float("nan"))
            out = tvg.dwconv2d_fused(x, d["w"], d["scale"], d["shift"], d["bias"], r, stride=stride,
                                     pad=1, relu=relu, stream_out=hint, out=y)
            torch.cuda.synchronize()
            assert out.data_ptr() == y.data_ptr()
            check(to_host(y), want, dtype, (cfg, variant, off, hint))


@pytest.mark.parametrize("i", [0, 2, 3, 4, 5, 6, 7, 8])
def test_depthwise_batch64_full(tvg, i):
    """D1, D3..D9 at batch 64 (HBM-sized traffic): the launch configuration of the
    supplementary bandwidth measurement, every output against the oracle."""
    import torch
    sh = ti.mobilenet_depthwise(64)[i]
    inp = ti.make_inputs(sh, ti.layer_seed(3, 100 + i), "f32")
    d = dev_inputs(inp, "f32")
    y = tvg.dwconv2d_fused(d["x"], d["w"], d["scale"], d["shift"], stride=sh.stride, pad=1,
                           relu=True, stream_out=True)       # as bench.py launches it
    plain = tvg.dwconv2d_fused(d["x"], d["w"], d["scale"], d["shift"], stride=sh.stride, pad=1,
                               relu=True)
    torch.cuda.synchronize()
    assert torch.equal(y, plain)                  # the store hint changes no value
    want = oracle.dwconv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"],
                                 stride=(sh.stride,) * 2, pad=(1, 1), relu=True)
    check(to_host(y), want, "f32", sh.name)


# ------------------------------------------------------------------------------------------
# dense conv
# ------------------------------------------------------------------------------------------

def test_config1_single_conv_fp32(tvg):
    sh = ti.config1_shape()
    inp = ti.make_inputs(sh, ti.layer_seed(1, 0), "f32")
    y = run_dense(tvg, sh, inp, "f32")
    check(to_host(y), oracle_dense(sh, inp), "f32")


@pytest.mark.parametrize("i", range(12))
def test_config2_resnet18_shapes_fp32_batch1(tvg, i):
    sh = ti.resnet18_convs(1)[i]
    inp = ti.make_inputs(sh, ti.layer_seed(2, i), "f32")
    y = run_dense(tvg, sh, inp, "f32")
    assert tuple(y.shape) == sh.y_shape()
    check(to_host(y), oracle_dense(sh, inp), "f32")


RAGGED = [
    # n, ic, h, w, oc, r, s, stride, pad
    (1, 3, 17, 19, 5, 3, 3, 1, 1),
    (3, 3, 23, 21, 40, 7, 7, 2, 3),
    (2, 17, 9, 9, 33, 1, 1, 1, 0),
    (2, 20, 15, 13, 70, 1, 1, 2, 0),
    (3, 5, 12, 14, 130, 3, 3, 2, 1),
    (1, 64, 7, 7, 200, 3, 3, 1, 1),
    (2, 9, 11, 10, 6, 5, 5, 1, 2),          # filter size without a specialised instance
    (1, 1, 3, 3, 1, 3, 3, 1, 1),
    (5, 48, 6, 6, 96, 3, 3, 1, 0),          # no padding
    (1, 260, 5, 5, 64, 3, 3, 1, 1),         # long reduction with a ragged last chunk
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cfg", RAGGED)
def test_dense_ragged_shapes_full_tail(tvg, dtype, cfg):
    n, ic, h, w, oc, r, s, stride, pad = cfg
    sh = ti.ConvShape("x", n, ic, h, w, oc, r, s, stride, pad)
    inp = ti.make_inputs(sh, 777 + sum(cfg), dtype, residual=True, bias=True)
    y = run_dense(tvg, sh, inp, dtype)
    check(to_host(y), oracle_dense(sh, inp), dtype)


PATCH_RAGGED = [
    # bf16 3x3 pad-1 problems with IC % 16 == 0: n, ic, h, w, oc, stride
    (3, 16, 9, 11, 40, 1), (2, 32, 10, 13, 70, 2), (5, 48, 7, 7, 130, 1), (4, 16, 5, 6, 8, 2),
    (1, 64, 1, 1, 64, 1), (2, 16, 2, 3, 16, 2), (1, 16, 30, 70, 16, 1), (1, 16, 33, 120, 200, 2),
    (7, 32, 7, 7, 64, 2), (2, 16, 14, 14, 256, 1), (3, 16, 56, 56, 64, 1), (2, 16, 57, 55, 32, 2),
    # stride 2 with rows that take 8-byte and 16-byte loads (W % 4 == 0, W % 8 == 0): even and
    # odd columns are stored apart, several images per tile, ragged tails
    (2, 32, 28, 28, 96, 2), (3, 16, 12, 12, 40, 2), (1, 48, 20, 36, 64, 2), (2, 16, 16, 24, 64, 2),
    (5, 16, 9, 8, 33, 2), (9, 32, 4, 4, 64, 2),
    # rows that are even but no multiple of the load: the last task of a row is short, and the
    # last load of the tensor reaches past its end
    (3, 32, 14, 14, 64, 2), (2, 16, 10, 10, 40, 2), (1, 16, 9, 18, 64, 2), (2, 16, 6, 22, 33, 2),
    (1, 16, 3, 6, 8, 1), (64, 32, 14, 14, 64, 2),
]


@pytest.mark.parametrize("tile", ["", "64,512", "64,256", "128,128", "128,64", "64,128", "64,64"])
@pytest.mark.parametrize("cfg", PATCH_RAGGED)
def test_bf16_3x3_patch_kernel_ragged_shapes_all_tiles(tvg, cfg, tile):
    """The LDS-patch 3x3 kernel under every workgroup tile shape it is built with (fixed through
    tvg_conv2d_set_tile; a shape the kernel cannot use falls back to the generic kernel)."""
    n, ic, h, w, oc, stride = cfg
    sh = ti.ConvShape("p", n, ic, h, w, oc, 3, 3, stride, 1)
    inp = ti.make_inputs(sh, 4000 + sum(cfg), "bf16", residual=True, bias=True)
    y = run_dense(tvg, sh, inp, "bf16", tile=tile)
    check(to_host(y), oracle_dense(sh, inp), "bf16")


WIDE_TILE_SHAPES = [
    # the single-stage kernel's 64 x 512 tile (stride 1, rows of 8n pixels): n, ic, h, w, oc
    (3, 64, 16, 24, 64), (2, 32, 8, 8, 130), (1, 16, 40, 64, 64), (5, 96, 24, 16, 72),
    (4, 64, 56, 56, 64), (1, 112, 3, 8, 40), (9, 64, 8, 8, 64), (2, 256, 16, 16, 64),
]


@pytest.mark.parametrize("cfg", WIDE_TILE_SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_bf16_3x3_patch_kernel_wide_tile(tvg, cfg):
    """64 x 512 tiles (one wave covers 64 channels x 128 pixels), fixed by tvg_conv2d_set_tile:
    the plan must really be that tile; bias, residual, ReLU; tiles that span several images,
    ragged channel and pixel tails."""
    n, ic, h, w, oc = cfg
    sh = ti.ConvShape("wt", n, ic, h, w, oc, 3, 3, 1, 1)
    desc = tvg.ConvDesc(n, ic, h, w, oc, 3, 3, 1, 1, 1, 1, tvg.TVG_BF16, 0)
    inp = ti.make_inputs(sh, 18000 + sum(cfg), "bf16", residual=True, bias=True)
    with fixed_tile(tvg, sh, "bf16", "64,512"):
        assert tvg.tvg_conv2d_get_plan(desc) == (1, 64, 512)
        y = run_dense(tvg, sh, inp, "bf16")
    check(to_host(y), oracle_dense(sh, inp), "bf16", cfg)


def test_bf16_3x3_wide_tile_is_the_rule_for_shallow_layers_that_fill_the_chip(tvg):
    def plan(n, ic, h, w, oc, stride=1):
        # (row_loads = 1, which even rows do not have: the rule of the kernels behind the kernel of strips)
        desc = tvg.ConvDesc(n, ic, h, w, oc, 3, 3, stride, stride, 1, 1, tvg.TVG_BF16, 0)
        assert tvg.tvg_conv2d_set_knobs(desc, (0, 0, 0, 0, 0, 1)) == 0
        got = tvg.tvg_conv2d_get_plan(desc)
        tvg.tvg_conv2d_set_knobs(desc, None)
        return got
    assert plan(64, 64, 56, 56, 64) == (1, 64, 512)        # C2 at batch 64: 392 tiles
    assert plan(32, 64, 56, 56, 64) == (1, 64, 256)        # batch 32: the wide tile would leave CUs idle
    assert plan(64, 128, 28, 28, 128) == (2, 64, 256)      # eight chunks: the pipelined kernel
    assert plan(64, 64, 56, 56, 128, 2)[2] != 512          # stride 2


DBUF_SHAPES = [
    # bf16 3x3 pad-1 stride-1 problems with IC % 32 == 0 and IC >= 128 (the software-pipelined
    # kernel): n, ic, h, w, oc.  Row lengths that are multiples of 8, 4, 2 and odd (16- to
    # 2-byte loads), images smaller than a tile, ragged channel and pixel tails, one-pixel rows.
    (1, 128, 1, 1, 64), (3, 128, 7, 7, 130), (2, 160, 9, 11, 40), (1, 128, 30, 70, 16),
    (2, 128, 8, 8, 64), (5, 192, 12, 12, 96), (1, 256, 33, 40, 72), (40, 128, 7, 7, 64),
    (2, 128, 3, 1, 64), (1, 128, 2, 64, 200), (3, 128, 5, 6, 8), (1, 512, 7, 7, 64),
    (2, 128, 56, 56, 64), (70, 128, 3, 3, 64),
    # rows of 4m + 2 pixels: 8-byte loads whose last task of a row is short
    (2, 128, 14, 14, 64), (3, 128, 10, 10, 96), (1, 256, 9, 22, 72),
]


@pytest.mark.parametrize("tile", ["", "64,256", "64,128", "64,64"])
@pytest.mark.parametrize("cfg", DBUF_SHAPES)
def test_bf16_3x3_pipelined_kernel_shapes_all_tiles(tvg, cfg, tile):
    """The two-stage 3x3 kernel under every pixel-tile width, with bias, residual and ReLU."""
    n, ic, h, w, oc = cfg
    sh = ti.ConvShape("db3", n, ic, h, w, oc, 3, 3, 1, 1)
    inp = ti.make_inputs(sh, 12000 + sum(cfg), "bf16", residual=True, bias=True)
    y = run_dense(tvg, sh, inp, "bf16", tile=tile)
    check(to_host(y), oracle_dense(sh, inp), "bf16")


DBUF_STRIDE2 = [
    # stride 2 under the pipelined kernel (IC % 32 == 0, IC >= 128, at most one workgroup per
    # CU): rows that take 4-, 8- and 16-byte loads, several images per tile, ragged tails
    (2, 128, 14, 14, 64), (3, 128, 9, 10, 130), (1, 256, 28, 28, 72), (2, 128, 16, 16, 64),
    (5, 160, 7, 8, 40), (1, 128, 2, 2, 64), (4, 128, 6, 12, 64), (64, 256, 14, 14, 64),
]


@pytest.mark.parametrize("tile", ["", "64,256", "64,128"])
@pytest.mark.parametrize("cfg", DBUF_STRIDE2)
def test_bf16_3x3_pipelined_kernel_stride2(tvg, cfg, tile):
    n, ic, h, w, oc = cfg
    sh = ti.ConvShape("db2", n, ic, h, w, oc, 3, 3, 2, 1)
    inp = ti.make_inputs(sh, 7100 + sum(cfg), "bf16", residual=True, bias=True)
    y = run_dense(tvg, sh, inp, "bf16", tile=tile)
    check(to_host(y), oracle_dense(sh, inp), "bf16")


KNOB_SHAPES = [
    # bf16 3x3 stride-1 problems for the pipelined kernel's knobs (input channels a multiple of
    # 64 so that two wave groups can split the reduction): n, ic, h, w, oc
    (3, 128, 7, 7, 130), (40, 128, 7, 7, 64), (1, 512, 7, 7, 64), (70, 128, 3, 3, 64),
    (2, 128, 3, 1, 64), (9, 192, 5, 5, 96), (2, 256, 14, 14, 72), (1, 128, 30, 70, 16),
    (5, 192, 12, 12, 96), (2, 128, 9, 11, 40), (1, 64, 7, 7, 64), (33, 256, 7, 5, 200),
]
KNOB_POINTS = [
    # (tile, split_k, lds_pitch, row_loads); stages = 2 throughout
    ("64,128", 2, 1, 1), ("64,128", 2, 2, 1), ("64,256", 2, 1, 1), ("64,256", 1, 2, 1),
    ("64,128", 1, 1, 2), ("64,128", 2, 1, 2), ("64,256", 2, 2, 2), ("64,64", 1, 2, 2),
]


@pytest.mark.parametrize("point", KNOB_POINTS, ids=lambda p: f"{p[0]}-k{p[1]}-p{p[2]}-r{p[3]}")
@pytest.mark.parametrize("cfg", KNOB_SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_bf16_3x3_pipelined_kernel_knobs(tvg, cfg, point):
    """The pipelined kernel under its knobs, fixed through tvg_conv2d_set_knobs: two wave groups
    splitting the reduction, both LDS pitches, whole-row loads of odd rows (start addresses of
    both parities, rows of 1 to 7 pixels).  A point the problem cannot use (the library would run
    something else) is skipped; what runs is checked against the oracle with bias, residual, ReLU."""
    import torch
    n, ic, h, w, oc = cfg
    tile, split_k, pitch, rows = point
    mt, nt = (int(v) for v in tile.split(","))
    sh = ti.ConvShape("kn", n, ic, h, w, oc, 3, 3, 1, 1)
    desc = tvg.ConvDesc(n, ic, h, w, oc, 3, 3, 1, 1, 1, 1, tvg.TVG_BF16, 0)
    want_knobs = (mt, nt, 2, split_k, pitch, rows if (w % 2 == 1 and w <= 7) else 0)
    assert tvg.tvg_conv2d_set_knobs(desc, want_knobs) == 0
    try:
        got_knobs = tvg.tvg_conv2d_get_knobs(desc)
        if tvg.tvg_conv2d_get_plan(desc)[0] != 2 or any(a and a != b for a, b in zip(want_knobs, got_knobs)):
            pytest.skip(f"point not usable here: asked {want_knobs}, would run {got_knobs}")
        inp = ti.make_inputs(sh, 15000 + sum(cfg) + split_k + 2 * pitch + 4 * rows, "bf16", residual=True, bias=True)
        y1 = run_dense(tvg, sh, inp, "bf16")
        y2 = run_dense(tvg, sh, inp, "bf16")
        assert torch.equal(y1.view(torch.int16), y2.view(torch.int16))      # deterministic
        check(to_host(y1), oracle_dense(sh, inp), "bf16", (cfg, got_knobs))
    finally:
        tvg.tvg_conv2d_set_knobs(desc, None)


MG_SHAPES = [
    # the pipelined kernel's channel-split variant (128-channel tiles, two wave groups that share
    # one patch): n, ic, h, w, oc, stride.  More than 64 output channels, at most 256 tiles; ragged
    # channel tails in the second group (130, 72, 200), several images per tile, every load width,
    # both strides, the full C6, C7 and C10 launches of the benchmark.
    (2, 128, 8, 8, 128, 1), (3, 128, 7, 7, 130, 1), (1, 256, 33, 40, 72, 1), (5, 192, 12, 12, 96, 1),
    (2, 128, 56, 56, 128, 1), (1, 128, 30, 70, 200, 1), (40, 128, 7, 7, 128, 1), (2, 128, 14, 14, 256, 1),
    (1, 128, 2, 64, 200, 1), (2, 128, 3, 1, 128, 1), (3, 128, 10, 10, 96, 1), (64, 128, 28, 28, 128, 1),
    (2, 128, 14, 14, 128, 2), (3, 128, 9, 10, 130, 2), (1, 256, 28, 28, 72, 2), (2, 128, 16, 16, 128, 2),
    (5, 160, 7, 8, 72, 2), (4, 128, 6, 12, 128, 2), (64, 128, 28, 28, 256, 2), (64, 256, 14, 14, 512, 2),
]


@pytest.mark.parametrize("pitch", [1, 2])
@pytest.mark.parametrize("nt", [256, 128])
@pytest.mark.parametrize("cfg", MG_SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_bf16_3x3_pipelined_kernel_channel_split(tvg, cfg, nt, pitch):
    """128 x nt tiles of the pipelined kernel, fixed through tvg_conv2d_set_knobs; skipped where the
    library would not run that variant (too many tiles, a patch that does not fit); what runs is
    checked against the oracle with bias, residual and ReLU, and is deterministic."""
    import torch
    n, ic, h, w, oc, stride = cfg
    if stride == 2 and pitch == 1:
        pytest.skip("stride 2 has one pitch rule")
    sh = ti.ConvShape("mg", n, ic, h, w, oc, 3, 3, stride, 1)
    desc = tvg.ConvDesc(n, ic, h, w, oc, 3, 3, stride, stride, 1, 1, tvg.TVG_BF16, 0)
    want = (128, nt, 2, 0, pitch if stride == 1 else 0, 0)
    assert tvg.tvg_conv2d_set_knobs(desc, want) == 0
    try:
        got = tvg.tvg_conv2d_get_knobs(desc)
        if tvg.tvg_conv2d_get_plan(desc) != (2, 128, nt) or any(a and a != b for a, b in zip(want, got)):
            pytest.skip(f"variant not usable here: asked {want}, would run {got}")
        inp = ti.make_inputs(sh, 16000 + sum(cfg) + nt + pitch, "bf16", residual=True, bias=True)
        y1 = run_dense(tvg, sh, inp, "bf16")
        y2 = run_dense(tvg, sh, inp, "bf16", stream_out=True)
        assert torch.equal(y1.view(torch.int16), y2.view(torch.int16))
        check(to_host(y1), oracle_dense(sh, inp), "bf16", (cfg, got))
    finally:
        tvg.tvg_conv2d_set_knobs(desc, None)


@pytest.mark.parametrize("cfg", [(2, 128, 8, 8, 64), (3, 128, 7, 7, 130), (1, 256, 33, 40, 72)])
def test_bf16_3x3_pipelined_kernel_plain_tail_and_determinism(tvg, cfg):
    """No bias, no residual, no ReLU (negative outputs survive), and bit-identical reruns."""
    n, ic, h, w, oc = cfg
    sh = ti.ConvShape("db3", n, ic, h, w, oc, 3, 3, 1, 1)
    inp = ti.make_inputs(sh, 13000 + sum(cfg), "bf16", residual=False, bias=False)
    y1 = to_host(run_dense(tvg, sh, inp, "bf16", relu=False))
    y2 = to_host(run_dense(tvg, sh, inp, "bf16", relu=False))
    assert np.array_equal(y1, y2)
    check(y1, oracle_dense(sh, inp, relu=False), "bf16")
    assert (y1 < 0).any()


PATCH_WIDE = [
    # bf16 3x3 pad-1 problems with 64 or more input channels: n, ic, h, w, oc, stride
    (2, 64, 9, 11, 40, 1), (3, 64, 10, 13, 70, 2), (5, 96, 7, 7, 130, 1), (2, 128, 14, 14, 256, 1),
    (1, 64, 30, 70, 16, 1), (2, 64, 33, 40, 200, 2), (7, 64, 7, 7, 64, 2), (1, 64, 1, 1, 64, 1),
    (3, 80, 5, 6, 8, 2), (40, 64, 7, 7, 64, 1), (2, 64, 56, 56, 64, 1), (9, 128, 28, 28, 128, 1),
]


@pytest.mark.parametrize("tile", ["", "64,256", "128,128", "64,128", "64,64"])
@pytest.mark.parametrize("cfg", PATCH_WIDE)
def test_bf16_3x3_patch_kernel_many_chunks(tvg, cfg, tile):
    """The 3x3 patch kernel with several channel chunks per tile: tiles that straddle images,
    ragged channel and pixel tails, every tile shape."""
    n, ic, h, w, oc, stride = cfg
    sh = ti.ConvShape("pw3", n, ic, h, w, oc, 3, 3, stride, 1)
    inp = ti.make_inputs(sh, 9000 + sum(cfg), "bf16", residual=True, bias=True)
    y = run_dense(tvg, sh, inp, "bf16", tile=tile)
    check(to_host(y), oracle_dense(sh, inp), "bf16")


STEM_SHAPES = [
    # bf16 7x7 stride-2 pad-3 problems with few input channels: n, ic, h, w, oc
    (2, 3, 32, 32, 64), (3, 3, 40, 24, 70), (1, 4, 16, 16, 8), (5, 3, 18, 8, 64),
    (2, 1, 64, 64, 16), (1, 3, 224, 224, 64), (2, 2, 50, 48, 100), (3, 3, 31, 40, 33),
    # an odd number of weights: the tensor ends in the middle of a 4-byte word
    (1, 1, 12, 48, 33), (3, 1, 34, 40, 33), (2, 3, 9, 16, 1),
]


@pytest.mark.parametrize("cfg", STEM_SHAPES)
def test_bf16_7x7_stem_kernel_shapes(tvg, cfg):
    """The stem kernel (and, for shapes it declines, its fallback) with the full fused tail."""
    n, ic, h, w, oc = cfg
    sh = ti.ConvShape("stem", n, ic, h, w, oc, 7, 7, 2, 3)
    inp = ti.make_inputs(sh, 6000 + sum(cfg), "bf16", residual=True, bias=True)
    y = run_dense(tvg, sh, inp, "bf16")
    check(to_host(y), oracle_dense(sh, inp), "bf16")


@pytest.mark.parametrize("cfg", STEM_SHAPES + [(32, 3, 224, 224, 32), (2, 3, 16, 16, 32), (4, 4, 10, 8, 40),
                                               # the 32-channel tile: ragged and tiny channel counts
                                               (3, 3, 64, 96, 24), (2, 3, 48, 40, 17), (1, 3, 224, 224, 1)])
def test_bf16_3x3_stride2_stem_kernel_shapes(tvg, cfg):
    """The same kernel with a 3x3 filter (pad 1): the MobileNet stem, 3 -> 32 channels, and the
    7x7 list's shapes; full fused tail; the plan must name the stem kernel for the large maps."""
    n, ic, h, w, oc = cfg
    sh = ti.ConvShape("stem3", n, ic, h, w, oc, 3, 3, 2, 1)
    desc = tvg.ConvDesc(n, ic, h, w, oc, 3, 3, 2, 2, 1, 1, tvg.TVG_BF16, 0)
    if cfg in ((32, 3, 224, 224, 32), (1, 3, 224, 224, 64), (2, 3, 32, 32, 64), (2, 1, 64, 64, 16),
               (3, 3, 64, 96, 24)):
        assert tvg.tvg_conv2d_get_plan(desc)[0] == 3      # (small maps may be declined: tiles that span images)
        assert tvg.tvg_conv2d_get_plan(desc)[1] == (32 if ic == 3 and oc <= 32 else 64)
    inp = ti.make_inputs(sh, 6500 + sum(cfg), "bf16", residual=True, bias=True)
    y = run_dense(tvg, sh, inp, "bf16")
    check(to_host(y), oracle_dense(sh, inp), "bf16", cfg)


PW_SHAPES = [
    # bf16 1x1 problems with IC % 8 == 0: n, ic, h, w, oc, stride
    (2, 8, 9, 9, 33, 1), (3, 40, 15, 13, 70, 2), (1, 64, 56, 56, 64, 1), (2, 72, 7, 7, 130, 1),
    (5, 16, 6, 10, 8, 2), (1, 264, 3, 5, 200, 1), (4, 32, 28, 28, 256, 2), (1, 8, 1, 1, 1, 1),
    # exactly 2 and 8 chunks of 32 channels (all chunks fetched up front), ragged tiles
    (3, 256, 14, 14, 130, 2), (2, 256, 9, 11, 70, 1), (20, 256, 14, 14, 512, 2), (3, 64, 13, 9, 40, 2),
    (2, 128, 10, 10, 96, 1),
    # map sizes and row lengths that are multiples of 8, 4 and 2, one and several chunks, ragged
    # channel tails
    (2, 64, 16, 16, 96, 2), (1, 96, 8, 24, 64, 2), (1, 40, 5, 6, 33, 1), (3, 200, 4, 8, 130, 1),
    (2, 64, 12, 28, 64, 2), (5, 32, 2, 4, 16, 2), (1, 256, 8, 8, 200, 1),
]


@pytest.mark.parametrize("cfg", PW_SHAPES)
def test_bf16_1x1_kernel_shapes(tvg, cfg):
    n, ic, h, w, oc, stride = cfg
    sh = ti.ConvShape("pw", n, ic, h, w, oc, 1, 1, stride, 0)
    inp = ti.make_inputs(sh, 8000 + sum(cfg), "bf16", residual=True, bias=True)
    y = run_dense(tvg, sh, inp, "bf16")
    check(to_host(y), oracle_dense(sh, inp), "bf16")


# n, ic, h, w, oc, stride: reductions of 4, 6, 8, 12, 16, 20 and 32 chunks of 32 channels (whole
# reduction fetched up front: 4 and 8; the rolling window of four - two under the 128 x 128 tile -
# otherwise), ragged channel and pixel tails, 7x7 maps, under each of the four tiles
PW_WINDOW_SHAPES = [(2, 128, 9, 9, 70, 1), (3, 192, 7, 7, 130, 1), (2, 256, 10, 6, 96, 2),
                    (1, 384, 14, 14, 200, 1), (2, 512, 14, 14, 512, 1), (3, 512, 7, 7, 72, 2),
                    (1, 640, 8, 9, 40, 1), (2, 1024, 7, 7, 130, 1), (33, 512, 2, 2, 64, 1)]


@pytest.mark.parametrize("tile", [(64, 64), (128, 64), (64, 128), (128, 128)], ids=lambda t: f"{t[0]}x{t[1]}")
@pytest.mark.parametrize("cfg", PW_WINDOW_SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_bf16_1x1_kernel_chunk_windows_all_tiles(tvg, cfg, tile):
    n, ic, h, w, oc, stride = cfg
    sh = ti.ConvShape("pw", n, ic, h, w, oc, 1, 1, stride, 0)
    desc = tvg.ConvDesc(n, ic, h, w, oc, 1, 1, stride, stride, 0, 0, tvg.TVG_BF16, 0)
    if tile[0] == 128 and oc <= 64:
        pytest.skip("no 128-channel tile for layers of at most 64 channels")
    assert tvg.tvg_conv2d_set_knobs(desc, (tile[0], tile[1], 0, 0, 0, 0)) == 0
    try:
        assert tvg.tvg_conv2d_get_plan(desc) == (4, tile[0], tile[1])
        inp = ti.make_inputs(sh, 8800 + sum(cfg) + tile[0] + tile[1], "bf16", residual=True, bias=True)
        y = run_dense(tvg, sh, inp, "bf16")
        check(to_host(y), oracle_dense(sh, inp), "bf16", (cfg, tile))
    finally:
        tvg.tvg_conv2d_set_knobs(desc, None)


DEEP_PW_SHAPES = [
    # bf16 1x1 stride-1 problems with IC % 128 == 0 and maps of 4n pixels (the deep-reduction
    # pointwise kernel): n, ic, h, w, oc.  16- and 8-byte pixel loads (HW % 8 == 0 or not), 2 to 16
    # steps, ragged channel and pixel tails, tiles that span several images, the MobileNet layers.
    (2, 512, 14, 14, 512), (3, 128, 4, 4, 64), (1, 256, 6, 6, 72), (2, 1024, 2, 2, 130),
    (5, 256, 28, 28, 256), (1, 384, 10, 10, 200), (2, 128, 56, 56, 128), (3, 256, 2, 2, 64),
    (1, 128, 4, 1, 64), (70, 256, 2, 2, 64), (32, 512, 14, 14, 512), (2, 2048, 2, 6, 96),
    (1, 640, 8, 9, 40),
]


@pytest.mark.parametrize("variant", ["plain", "bias+residual", "no-relu"])
@pytest.mark.parametrize("cfg", DEEP_PW_SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_bf16_1x1_deep_kernel_shapes(tvg, cfg, variant):
    """The deep-reduction pointwise kernel, named through the stages knob (no rule picks it): every
    output against the oracle, deterministic, hint-independent."""
    import torch
    n, ic, h, w, oc = cfg
    sh = ti.ConvShape("pwd", n, ic, h, w, oc, 1, 1, 1, 0)
    desc = tvg.ConvDesc(n, ic, h, w, oc, 1, 1, 1, 1, 0, 0, tvg.TVG_BF16, 0)
    assert tvg.tvg_conv2d_set_knobs(desc, (0, 0, 2, 0, 0, 0)) == 0
    try:
        assert tvg.tvg_conv2d_get_plan(desc) == (6, 64, 128)
        inp = ti.make_inputs(sh, 17000 + sum(cfg) + len(variant), "bf16", residual="residual" in variant,
                             bias="bias" in variant)
        relu = "no-relu" not in variant
        y1 = run_dense(tvg, sh, inp, "bf16", relu=relu)
        y2 = run_dense(tvg, sh, inp, "bf16", relu=relu, stream_out=True)
        assert torch.equal(y1.view(torch.int16), y2.view(torch.int16))
        check(to_host(y1), oracle_dense(sh, inp, relu=relu), "bf16", (cfg, variant))
        # the general pointwise kernel on the same problem (stages = 1): same operator
        assert tvg.tvg_conv2d_set_knobs(desc, (0, 0, 1, 0, 0, 0)) == 0
        assert tvg.tvg_conv2d_get_plan(desc)[0] == 4
        y3 = run_dense(tvg, sh, inp, "bf16", relu=relu)
        check(to_host(y3), oracle_dense(sh, inp, relu=relu), "bf16", (cfg, variant, "general"))
    finally:
        tvg.tvg_conv2d_set_knobs(desc, None)


def test_bf16_1x1_kernel_unaligned_input(tvg):
    """x at an 8-byte and at a 2-byte offset from an aligned address (the kernel needs 2-byte
    alignment only)."""
    import torch
    sh = ti.ConvShape("pwa", 2, 64, 8, 8, 64, 1, 1, 1, 0)
    inp = ti.make_inputs(sh, 8123, "bf16")
    d = dev_inputs(inp, "bf16")
    want = oracle_dense(sh, inp)
    for off in (4, 1):
        store = torch.empty(d["x"].numel() + 16, dtype=torch.bfloat16, device="cuda:0")
        x = store[off:off + d["x"].numel()].view(d["x"].shape)
        x.copy_(d["x"])
        y = tvg.conv2d_fused(x, d["w"], d["scale"], d["shift"], stride=1, pad=0, relu=True)
        torch.cuda.synchronize()
        check(to_host(y), want, "bf16", off)


F32_SMALL = [
    # fp32 launch-bound problems for the one-launch kernel (1x1 / 3x3, "same" padding, input
    # channels a multiple of 8): n, ic, h, w, oc, k, stride.  Rows of 4n pixels (16-byte copies)
    # and others, 1 to 16 waves per workgroup, one and several passes, ragged channel and pixel
    # tails, tiles at the top and bottom image borders, several images.
    (1, 64, 56, 56, 64, 3, 1), (1, 64, 56, 56, 128, 3, 2), (1, 128, 28, 28, 128, 3, 1),
    (1, 256, 14, 14, 512, 3, 2), (1, 512, 7, 7, 512, 3, 1), (1, 64, 56, 56, 64, 1, 1),
    (1, 256, 14, 14, 512, 1, 2), (2, 8, 9, 11, 33, 3, 1), (3, 24, 5, 6, 70, 3, 2),
    (1, 40, 1, 1, 5, 3, 1), (2, 16, 12, 8, 40, 1, 1), (1, 136, 7, 9, 64, 3, 1),
    (2, 1024, 7, 7, 48, 1, 1), (1, 32, 30, 64, 16, 3, 1), (3, 48, 13, 16, 130, 3, 2),
    (1, 8, 2, 3, 1, 1, 2), (4, 64, 4, 4, 96, 3, 1), (1, 16, 33, 4, 8, 3, 1),
]


@pytest.mark.parametrize("cfg", F32_SMALL, ids=lambda c: "x".join(map(str, c)))
def test_fp32_small_kernel_shapes(tvg, cfg):
    n, ic, h, w, oc, k, stride = cfg
    sh = ti.ConvShape("f32s", n, ic, h, w, oc, k, k, stride, k // 2)
    desc = tvg.ConvDesc(n, ic, h, w, oc, k, k, stride, stride, k // 2, k // 2, tvg.TVG_F32, 0)
    assert tvg.tvg_conv2d_get_plan(desc)[0] == 5, "expected the fp32 kernel for launch-bound problems"
    inp = ti.make_inputs(sh, 17000 + sum(cfg), "f32", residual=True, bias=True)
    y1 = to_host(run_dense(tvg, sh, inp, "f32"))
    y2 = to_host(run_dense(tvg, sh, inp, "f32"))
    assert np.array_equal(y1, y2)                                # deterministic
    check(y1, oracle_dense(sh, inp), "f32", cfg)
    plain = ti.make_inputs(sh, 17500 + sum(cfg), "f32")
    y3 = to_host(run_dense(tvg, sh, plain, "f32", relu=False))
    check(y3, oracle_dense(sh, plain, relu=False), "f32", cfg)
    assert (y3 < 0).any()


F32_STEM = [
    # fp32 7x7 stride-2 pad-3 problems with at most four input channels and rows of 4n pixels (the
    # one-launch stem kernel of launch-bound problems): n, ic, h, w, oc
    (1, 3, 224, 224, 64), (2, 3, 32, 32, 64), (3, 1, 40, 24, 70), (1, 4, 16, 16, 8), (5, 3, 18, 8, 33),
    (2, 2, 50, 48, 100), (1, 3, 9, 12, 40), (2, 3, 64, 4, 32), (1, 3, 2, 4, 5), (1, 4, 31, 132, 64),
]


@pytest.mark.parametrize("variant", ["plain", "bias+residual", "no-relu"])
@pytest.mark.parametrize("cfg", F32_STEM, ids=lambda c: "x".join(map(str, c)))
def test_fp32_stem_kernel_shapes(tvg, cfg, variant):
    """Seven waves, one per filter row, partial tiles added through LDS: full fused tail, tiles that
    end in the middle of a row, maps smaller than a tile, channel tails."""
    n, ic, h, w, oc = cfg
    sh = ti.ConvShape("f32stem", n, ic, h, w, oc, 7, 7, 2, 3)
    desc = tvg.ConvDesc(n, ic, h, w, oc, 7, 7, 2, 2, 3, 3, tvg.TVG_F32, 0)
    assert tvg.tvg_conv2d_get_plan(desc)[0] == 5
    assert tvg.tvg_conv2d_workspace_size(desc) == 0
    inp = ti.make_inputs(sh, 19000 + sum(cfg) + len(variant), "f32", residual="residual" in variant,
                         bias="bias" in variant)
    relu = "no-relu" not in variant
    y = run_dense(tvg, sh, inp, "f32", relu=relu)
    check(to_host(y), oracle_dense(sh, inp, relu=relu), "f32", (cfg, variant))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rectangular_filter_and_strides(tvg, dtype):
    import torch
    rng = np.random.default_rng(99)
    x = rng.uniform(-1, 1, (2, 6, 13, 17)).astype(np.float32)
    w = rng.uniform(-1, 1, (10, 6, 5, 2)).astype(np.float32)
    if dtype == "bf16":
        x, w = ti.quantize_bf16(x), ti.quantize_bf16(w)
    scale = rng.uniform(0.5, 1.5, 10).astype(np.float32)
    shift = rng.uniform(-0.1, 0.1, 10).astype(np.float32)
    y = tvg.conv2d_fused(to_dev(x, dtype), to_dev(w, dtype), to_dev(scale, "f32"),
                         to_dev(shift, "f32"), stride=(2, 3), pad=(2, 1), relu=False)
    torch.cuda.synchronize()
    want = oracle.conv2d_fused(x, w, scale, shift, stride=(2, 3), pad=(2, 1), relu=False)
    check(to_host(y), want, dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_identity_kernel_is_bit_exact(tvg, dtype):
    import torch
    c = 96
    sh = ti.ConvShape("id", 2, c, 14, 14, c, 3, 3, 1, 1)
    x = ti.make_inputs(sh, 5, dtype)["x"]
    w = np.zeros(sh.w_shape(), np.float32)
    w[np.arange(c), np.arange(c), 1, 1] = 1.0
    y = tvg.conv2d_fused(to_dev(x, dtype), to_dev(w, dtype), to_dev(np.ones(c), "f32"),
                         to_dev(np.zeros(c), "f32"), stride=1, pad=1, relu=False)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(y), x.astype(np.float64))


def test_results_are_deterministic_and_stay_inside_y(tvg):
    """Run twice into NaN-filled buffers with guard bands: same bits, guards untouched."""
    import torch
    for sh, dtype in [(ti.resnet18_convs(1)[11], "f32"), (ti.resnet18_convs(2)[5], "bf16")]:
        inp = ti.make_inputs(sh, 31337, dtype, residual=True)
        d = dev_inputs(inp, dtype)
        numel = int(np.prod(sh.y_shape()))
        guard = 4096
        outs = []
        for _ in range(2):
            buf = torch.full((numel + 2 * guard,), float("nan"), dtype=d["x"].dtype, device="cuda")
            y = buf[guard:guard + numel].view(sh.y_shape())
            tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], None, d["residual"],
                             stride=sh.stride, pad=sh.pad, relu=True, out=y)
            torch.cuda.synchronize()
            assert torch.isnan(buf[:guard]).all() and torch.isnan(buf[guard + numel:]).all()
            assert not torch.isnan(y).any()
            outs.append(y.clone())
        assert torch.equal(outs[0], outs[1])


def test_output_may_alias_residual(tvg):
    import torch
    sh = ti.resnet18_convs(2)[1]
    inp = ti.make_inputs(sh, 2024, "bf16", residual=True)
    d = dev_inputs(inp, "bf16")
    y = d["residual"].clone()
    tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], None, y, stride=1, pad=1, relu=True,
                     out=y)
    torch.cuda.synchronize()
    check(to_host(y), oracle_dense(sh, inp), "bf16")


@pytest.mark.parametrize("i", range(12))
def test_config4_resnet18_shapes_bf16_batch64_full(tvg, i):
    """Full-size launch (the configuration bench.py times, store hint included): EVERY output
    of the layer against the oracle - all 64 images, every tile, image wrap and ragged tail -
    at the stated 2e-2 and at the tight one-rounding bound."""
    import torch
    sh = ti.resnet18_convs(64)[i]
    inp = ti.make_inputs(sh, ti.layer_seed(4, i), "bf16")
    y = run_dense(tvg, sh, inp, "bf16", stream_out=True)      # as bench.py launches it
    # the store hint changes no value: bit-identical to the plain launch
    assert torch.equal(y.view(torch.int16), run_dense(tvg, sh, inp, "bf16").view(torch.int16))
    got = to_host(y)
    assert tuple(got.shape) == sh.y_shape()
    check(got, oracle_dense(sh, inp), "bf16", sh.name)
    assert np.all(got >= 0)


# ------------------------------------------------------------------------------------------
# max-pool and the chained ResNet-18 body (configuration 5)
# ------------------------------------------------------------------------------------------

@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(2, 3, 8, 8), (1, 5, 7, 9), (2, 64, 112, 112), (1, 2, 1, 1),
                                   (3, 5, 9, 16), (1, 4, 2, 8), (2, 7, 13, 40), (1, 3, 1, 24)])
def test_maxpool_is_exact(tvg, dtype, shape):
    import torch
    rng = np.random.default_rng(sum(shape))
    x = rng.uniform(-1, 1, shape).astype(np.float32)
    if dtype == "bf16":
        x = ti.quantize_bf16(x)
    y = tvg.maxpool2d_3x3s2(to_dev(x, dtype))
    torch.cuda.synchronize()
    assert np.array_equal(to_host(y), oracle.maxpool2d(x))


def dual_params(weights, st):
    """Constant folding for a two-head step: the 3x3 filters of head 1 and the 1x1 filters of head 2
    (placed at the centre tap of zero 3x3 filters) as one weight tensor, scale and shift joined."""
    p1, p2 = weights[st.layer_index], weights[st.layer_index2]
    k2, c = p2["w"].shape[:2]
    emb = np.zeros((k2, c, 3, 3), np.float32)
    emb[:, :, 1, 1] = p2["w"][:, :, 0, 0]
    return {"w": np.concatenate([p1["w"], emb]), "scale": np.concatenate([p1["scale"], p2["scale"]]),
            "shift": np.concatenate([p1["shift"], p2["shift"]])}


def run_dual(tvg, st, src, p):
    """One tvg_conv2d_fused_dual launch for a "conv_dual" step; p = device tensors of dual_params."""
    import torch
    sh, s2 = st.shape, st.shape2
    desc = tvg.ConvDesc(sh.n, sh.ic, sh.h, sh.w, sh.oc + s2.oc, 3, 3, sh.stride, sh.stride, 1, 1,
                        tvg.TVG_BF16, tvg.TVG_RELU if st.relu else 0)
    y1 = torch.empty(sh.y_shape(), dtype=torch.bfloat16, device="cuda:0")
    y2 = torch.empty(s2.y_shape(), dtype=torch.bfloat16, device="cuda:0")
    flags2 = (tvg.TVG_RELU if st.relu2 else 0) | tvg.TVG_CENTRE_TAP_ONLY
    rc = tvg.tvg_conv2d_fused_dual(desc, sh.oc, flags2, src, p["w"], p["scale"], p["shift"], None, None, y1, y2)
    assert rc == 0, tvg.status_string(rc)
    return y1, y2


def run_body_gpu(tvg, steps, images, weights):
    import torch
    tensors = {0: to_dev(images, "bf16")}
    dev_w = {k: {n: to_dev(v, "bf16" if n == "w" else "f32") for n, v in p.items()}
             for k, p in weights.items()}
    for st in steps:
        src = tensors[st.src]
        if st.op == "conv_dual":
            p = {n: to_dev(v, "bf16" if n == "w" else "f32") for n, v in dual_params(weights, st).items()}
            tensors[st.dst], tensors[st.dst2] = run_dual(tvg, st, src, p)
        elif st.op == "conv":
            p = dev_w[st.layer_index]
            res = None if st.residual is None else tensors[st.residual]
            tensors[st.dst] = tvg.conv2d_fused(src, p["w"], p["scale"], p["shift"], None, res,
                                               stride=st.shape.stride, pad=st.shape.pad,
                                               relu=st.relu)
        elif st.op == "dwconv":
            p = dev_w[st.layer_index]
            tensors[st.dst] = tvg.dwconv2d_fused(src, p["w"], p["scale"], p["shift"], None, None,
                                                 stride=st.shape.stride, pad=st.shape.pad,
                                                 relu=st.relu)
        else:
            tensors[st.dst] = tvg.maxpool2d_3x3s2(src)
    torch.cuda.synchronize()
    return tensors


def body_weights(steps, config=5):
    return {s.layer_index: ti.make_weights(s.shape, ti.layer_seed(config, s.layer_index), "bf16")
            for s in steps if s.op in ("conv", "dwconv")}


def chain_drift(g, r):
    """(rms, worst element, signed mean in standard errors) of a chain's last tensor against the
    oracle chain's, all relative to the oracle tensor's RMS."""
    rho = float(np.sqrt(np.mean(r * r)))
    d = (g - r) / rho
    rms = float(np.sqrt(np.mean(d * d)))
    # Errors of neighbouring outputs share their inputs' flipped roundings, so the elements are
    # not independent samples: a 3x3 window over the last layers' channels correlates roughly
    # the 9 positions of a window; the standard error is taken over n / 9 samples.
    stderr = float(np.std(d)) / np.sqrt(d.size / 9.0)
    return rms, rel_err(g, r), float(np.mean(d)) / stderr


def test_config5_resnet18_body_bf16_small_batch_full(tvg):
    """The whole 21-launch chain at batch 2.

    THE GATE (per operator, the stated 2e-2, plus the tight one-rounding bound): every layer's
    complete output against the oracle fed with the GPU's own input of that layer.

    SUPPLEMENTARY, not the stated tolerance: the last tensor against the oracle chain (fp64
    per layer, outputs rounded to bf16 as stored).  Two correct bf16-storing chains that sum in
    different orders do not stay within one rounding of each other: a last-bit difference in
    one stored activation is a full bf16 ulp (2^-8 relative), after a few layers most elements
    differ by an ulp, and from then on each layer adds independent rounding noise of about
    0.16 % rms which the next convolution passes on undiminished relative to its output rms.
    Over 20 layers the two chains differ by about sqrt(2*20)*0.16 % = 1 % rms and a few sigma
    at the worst element, so this check bounds the rms-normalised error by 2e-2 and the worst
    element by 8e-2 (this test's own bounds, derived above), and requires the drift to be
    noise, not bias: the signed mean of (gpu - oracle)/rho within four standard errors of zero.
    """
    from oracle.resnet_body import run_steps
    steps = ti.resnet18_body(2)
    weights = body_weights(steps)
    images = ti.body_images(2, ti.layer_seed(5, 900))
    got = run_body_gpu(tvg, steps, images, weights)
    host = {k: v.float().cpu().numpy() for k, v in got.items()}
    for st in steps:
        if st.op == "maxpool":
            assert np.array_equal(host[st.dst].astype(np.float64), oracle.maxpool2d(host[st.src]))
            continue
        p = weights[st.layer_index]
        res = None if st.residual is None else host[st.residual]
        want = oracle.conv2d_fused(host[st.src], p["w"], p["scale"], p["shift"], None, res,
                                   stride=(st.shape.stride,) * 2, pad=(st.shape.pad,) * 2,
                                   relu=st.relu)
        check(host[st.dst], want, "bf16", st.name)
    want = run_steps(steps, images, weights)
    final = steps[-1].dst
    assert tuple(got[final].shape) == (2, 512, 7, 7)
    rms, worst, bias_se = chain_drift(to_host(got[final]), want[final].astype(np.float64))
    print(f"chain drift: rms {rms:.3e} worst {worst:.3e} signed mean {bias_se:+.2f} standard errors")
    assert rms <= 2e-2
    assert worst <= 8e-2
    assert abs(bias_se) <= 4.0


DUAL_SHAPES = [
    # n, c, h, w, k1, k2, stride: the ResNet-18 down-sampling blocks (C4+C5, C7+C8, C10+C11) and
    # ragged cases: pixel tails, a head 2 that is no multiple of the tile, odd maps, stride 1
    (2, 64, 56, 56, 128, 128, 2), (2, 128, 28, 28, 256, 256, 2), (3, 256, 14, 14, 512, 512, 2),
    (3, 16, 9, 11, 64, 40, 1), (2, 32, 10, 13, 128, 70, 2), (5, 48, 7, 7, 64, 1, 1),
    (1, 16, 30, 70, 192, 33, 2), (7, 32, 7, 7, 64, 64, 2), (2, 16, 2, 3, 64, 16, 2),
]


@pytest.mark.parametrize("centre_only", [True, False])
@pytest.mark.parametrize("cfg", DUAL_SHAPES, ids=lambda c: "x".join(map(str, c)))
def test_two_head_conv(tvg, cfg, centre_only):
    """tvg_conv2d_fused_dual: head 1 against the oracle's 3x3 convolution (bias, residual, ReLU),
    head 2 against the oracle's 1x1 convolution of the same input with the same stride (centre
    tap only) or against a full 3x3 convolution (no promise about the filters); bit-identical
    reruns."""
    import torch
    n, c, h, w, k1, k2, stride = cfg
    s1 = ti.ConvShape("h1", n, c, h, w, k1, 3, 3, stride, 1)
    s2 = ti.ConvShape("h2", n, c, h, w, k2, 1, 1, stride, 0) if centre_only else \
        ti.ConvShape("h2", n, c, h, w, k2, 3, 3, stride, 1)
    a = ti.make_inputs(s1, 19000 + sum(cfg), "bf16", residual=True, bias=True)
    b = ti.make_inputs(s2, 19500 + sum(cfg), "bf16", bias=True)
    w2 = b["w"]
    if centre_only:
        w2 = np.zeros((k2, c, 3, 3), np.float32)
        w2[:, :, 1, 1] = b["w"][:, :, 0, 0]
    cat = lambda u, v: np.concatenate([u, v])
    x = to_dev(a["x"], "bf16")
    dw, dsc, dsf, dbi = (to_dev(cat(a["w"], w2), "bf16"), to_dev(cat(a["scale"], b["scale"]), "f32"),
                         to_dev(cat(a["shift"], b["shift"]), "f32"), to_dev(cat(a["bias"], b["bias"]), "f32"))
    res = to_dev(a["residual"], "bf16")
    desc = tvg.ConvDesc(n, c, h, w, k1 + k2, 3, 3, stride, stride, 1, 1, tvg.TVG_BF16, tvg.TVG_RELU)
    outs = []
    for rep in range(2):
        y1 = torch.full(s1.y_shape(), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        y2 = torch.full(s2.y_shape(), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        rc = tvg.tvg_conv2d_fused_dual(desc, k1, tvg.TVG_CENTRE_TAP_ONLY if centre_only else 0, x, dw,
                                       dsc, dsf, dbi, res, y1, y2)
        assert rc == 0, tvg.status_string(rc)
        torch.cuda.synchronize()
        outs.append((y1, y2))
    assert torch.equal(outs[0][0].view(torch.int16), outs[1][0].view(torch.int16))
    assert torch.equal(outs[0][1].view(torch.int16), outs[1][1].view(torch.int16))
    a["x"] = b["x"] = a["x"]
    check(to_host(outs[0][0]), oracle_dense(s1, a), "bf16", ("head 1", cfg))
    b["x"] = a["x"]
    check(to_host(outs[0][1]), oracle_dense(s2, b, relu=False), "bf16", ("head 2", cfg))
    assert (to_host(outs[0][1]) < 0).any()


@pytest.mark.parametrize("batch", [2, 32])
def test_config5_resnet18_body_with_two_head_blocks(tvg, batch):
    """The ResNet-18 chain with each down-sampling block's first conv and projection shortcut as
    ONE two-head launch (18 launches): every tensor bit-identical to the 21-launch chain (the
    same products are summed in the same order), and, at the stated tolerance and the tight
    bound, every layer against the oracle fed with the GPU's own input of that layer."""
    import torch
    plain, fused = ti.resnet18_body(batch), ti.resnet18_body(batch, fuse_projection=True)
    weights = body_weights(plain)
    images = ti.body_images(batch, ti.layer_seed(5, 903))
    want = run_body_gpu(tvg, plain, images, weights)
    got = run_body_gpu(tvg, fused, images, weights)
    for k in want:
        same = torch.equal(got[k].view(torch.int16), want[k].view(torch.int16))
        assert same, f"tensor {k} differs between the fused and the plain chain"
    host = {k: v.float().cpu().numpy() for k, v in got.items()}
    del got, want
    for st in fused:
        if st.op != "conv_dual":
            continue
        for shape, lidx, dst, relu in ((st.shape, st.layer_index, st.dst, st.relu),
                                       (st.shape2, st.layer_index2, st.dst2, st.relu2)):
            p = weights[lidx]
            ref = oracle.conv2d_fused(host[st.src], p["w"], p["scale"], p["shift"], None, None,
                                      stride=(shape.stride,) * 2, pad=(shape.pad,) * 2, relu=relu)
            check(host[dst], ref, "bf16", (st.name, shape.name))


def test_tuner_fixes_a_tile_and_results_stay_right(tvg, tmp_path):
    """tune.tune_conv2d times the tile shapes of a problem through the C ABI and fixes the
    fastest; whatever it picks, the result still matches the oracle, and the choice survives
    a save / load round trip."""
    import torch
    from paper_1802_04799_amd import tune
    sh = ti.ConvShape("tn", 8, 64, 28, 28, 128, 3, 3, 1, 1)
    inp = ti.make_inputs(sh, 9911, "bf16")
    d = dev_inputs(inp, "bf16")
    desc = tvg.ConvDesc(sh.n, sh.ic, sh.h, sh.w, sh.oc, 3, 3, 1, 1, 1, 1, tvg.TVG_BF16, tvg.TVG_RELU)
    y = torch.empty(sh.y_shape(), dtype=torch.bfloat16, device="cuda:0")
    try:
        rep = tune.tune_conv2d(desc, d["x"], d["w"], d["scale"], d["shift"], y, iters=10, repeats=2,
                               min_gain=0.0, max_trials=12)
        assert rep["kernel"] == "3x3" and len(rep["candidates"]) >= 3
        assert rep["tuned_us"] <= rep["default_us"]
        walk = rep["walk"]
        assert 3 <= walk["trials"] <= 12 and walk["space_points"] > 12 and not walk["exhaustive"]
        plan = tvg.tvg_conv2d_get_plan(desc)
        if rep["chosen"]:
            assert list(plan[1:]) == rep["chosen"]
            assert all(w == 0 or w == g for w, g in zip(rep["chosen_knobs"], tvg.tvg_conv2d_get_knobs(desc)))
        out = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], stride=1, pad=1, relu=True)
        torch.cuda.synchronize()
        check(to_host(out), oracle_dense(sh, inp), "bf16")
        path = str(tmp_path / "tiles.json")
        tune.save(path)
        knobs = tvg.tvg_conv2d_get_knobs(desc)
        tvg.tvg_conv2d_set_knobs(desc, None)
        assert tune.load(path) == (1 if rep["chosen"] else 0)
        assert tvg.tvg_conv2d_get_plan(desc) == plan and tvg.tvg_conv2d_get_knobs(desc) == knobs
    finally:
        tvg.tvg_conv2d_set_knobs(desc, None)


def test_config5_resnet18_body_hip_graph_replays_match_eager(tvg):
    """The 21-launch chain recorded once into a HIP graph: the library allocates nothing and
    never synchronises, so it records as it stands.  Three replays, each on new images written
    into the captured input buffer, with eager launches and synchronisations between them;
    every tensor of every replay is bit-identical to the eager chain on the same images."""
    import torch
    steps = ti.resnet18_body(2)
    weights = body_weights(steps)
    dev_w = {k: {n: to_dev(v, "bf16" if n == "w" else "f32") for n, v in p.items()}
             for k, p in weights.items()}
    images = to_dev(ti.body_images(2, ti.layer_seed(5, 900)), "bf16")
    tensors, calls = {0: images}, []
    for st in steps:
        src = tensors[st.src]
        if st.op == "conv":
            sh, p = st.shape, dev_w[st.layer_index]
            desc = tvg.ConvDesc(sh.n, sh.ic, sh.h, sh.w, sh.oc, sh.r, sh.s, sh.stride, sh.stride,
                                sh.pad, sh.pad, tvg.TVG_BF16, tvg.TVG_RELU if st.relu else 0)
            y = torch.empty(sh.y_shape(), dtype=torch.bfloat16, device="cuda:0")
            need = tvg.tvg_conv2d_workspace_size(desc)
            ws = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda:0")
            res = None if st.residual is None else tensors[st.residual]
            calls.append((tvg.tvg_conv2d_fused, (desc, src, p["w"], p["scale"], p["shift"], None,
                                                 res, y, ws, need, None)))
        else:
            n, c, h, w = src.shape
            y = torch.empty((n, c, (h - 1) // 2 + 1, (w - 1) // 2 + 1), dtype=torch.bfloat16,
                            device="cuda:0")
            calls.append((tvg.tvg_maxpool2d_3x3s2, (n, c, h, w, tvg.TVG_BF16, src, y, None)))
        tensors[st.dst] = y

    def forward():          # stream=None: the binding launches on torch's current stream
        for fn, a in calls:
            assert fn(*a) == 0

    forward()               # one-time kernel attributes are set outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        forward()
    for rep in range(3):
        images.copy_(to_dev(ti.body_images(2, ti.layer_seed(5, 910 + rep)), "bf16"))
        forward()
        torch.cuda.synchronize()
        want = {k: t.clone() for k, t in tensors.items()}
        for k, t in tensors.items():
            if k != 0:
                t.fill_(float("nan"))       # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k, t in tensors.items():
            assert torch.equal(t.view(torch.int16), want[k].view(torch.int16)), (rep, k)


def test_config5_resnet18_body_bf16_batch32_teacher_forced(tvg):
    """Batch 32 (the benchmark's launch configuration).  Every layer's COMPLETE output against
    the oracle fed with the GPU's own input of that layer, at the stated 2e-2 and at the tight
    one-rounding bound; the max-pool bit for bit."""
    steps = ti.resnet18_body(32)
    weights = body_weights(steps)
    images = ti.body_images(32, ti.layer_seed(5, 901))
    got = run_body_gpu(tvg, steps, images, weights)
    host = {k: v.float().cpu().numpy() for k, v in got.items()}
    del got
    for st in steps:
        if st.op == "maxpool":
            assert np.array_equal(host[st.dst].astype(np.float64), oracle.maxpool2d(host[st.src]))
            continue
        p = weights[st.layer_index]
        res = None if st.residual is None else host[st.residual]
        want = oracle.conv2d_fused(host[st.src], p["w"], p["scale"], p["shift"], None, res,
                                   stride=(st.shape.stride,) * 2, pad=(st.shape.pad,) * 2,
                                   relu=st.relu)
        check(host[st.dst], want, "bf16", st.name)


def oracle_layer(st, host, weights, idx=None):
    p = weights[st.layer_index]
    kw = dict(stride=(st.shape.stride,) * 2, pad=(st.shape.pad,) * 2, relu=st.relu)
    if st.op == "dwconv":
        y = oracle.dwconv2d_fused(host[st.src], p["w"], p["scale"], p["shift"], None, None, **kw)
        return y if idx is None else y.reshape(-1)[idx]
    if idx is None:
        return oracle.conv2d_fused(host[st.src], p["w"], p["scale"], p["shift"], None, None, **kw)
    return oracle.conv2d_fused_at(host[st.src], p["w"], p["scale"], p["shift"], None, None,
                                  idx=idx, **kw)


def test_mobilenet_body_bf16_small_batch_full(tvg):
    """The 27-launch MobileNet body (stem, 13 x depthwise 3x3 + 1x1) at batch 2: every layer's
    complete output against the oracle fed with the GPU's own input of that layer (the gate:
    2e-2 and the tight bound), and, as a supplementary check, the last tensor against the
    oracle chain (fp64 per layer, stored as bf16) with the end-to-end bounds of the ResNet-18
    chain test scaled to 27 layers: rms 2.5e-2, worst element 1e-1, signed mean within four
    standard errors."""
    from oracle.resnet_body import run_steps
    steps = ti.mobilenet_body(2)
    weights = body_weights(steps, config=6)
    images = ti.body_images(2, ti.layer_seed(6, 900))
    got = run_body_gpu(tvg, steps, images, weights)
    host = {k: v.float().cpu().numpy() for k, v in got.items()}
    for st in steps:
        check(host[st.dst], oracle_layer(st, host, weights), "bf16", st.name)
    want = run_steps(steps, images, weights)
    final = steps[-1].dst
    assert tuple(got[final].shape) == (2, 1024, 7, 7)
    rms, worst, bias_se = chain_drift(to_host(got[final]), want[final].astype(np.float64))
    print(f"chain drift: rms {rms:.3e} worst {worst:.3e} signed mean {bias_se:+.2f} standard errors")
    assert rms <= 2.5e-2 and worst <= 1e-1           # supplementary, see the ResNet-18 chain test
    assert abs(bias_se) <= 4.0


def test_mobilenet_body_bf16_batch32_teacher_forced(tvg):
    """Batch 32, the launch configuration the benchmark times: every layer's complete output
    against the oracle fed with the GPU's own input of that layer."""
    steps = ti.mobilenet_body(32)
    weights = body_weights(steps, config=6)
    images = ti.body_images(32, ti.layer_seed(6, 901))
    got = run_body_gpu(tvg, steps, images, weights)
    host = {k: v.float().cpu().numpy() for k, v in got.items()}
    del got
    for st in steps:
        check(host[st.dst], oracle_layer(st, host, weights), "bf16", st.name)


# ------------------------------------------------------------------------------------------
# MobileNet block: depthwise 3x3 + 1x1 through tvg_dwpw_fused (one kernel where the map is
# small, two kernels otherwise)
# ------------------------------------------------------------------------------------------

def block_inputs(n, c, h, w, k, stride, dtype, seed, residual, bias):
    d = ti.ConvShape("bd", n, c, h, w, c, 3, 3, stride, 1, depthwise=True)
    p = ti.ConvShape("bp", n, c, d.oh, d.ow, k, 1, 1, 1, 0)
    a = ti.make_inputs(d, seed, dtype)
    b = ti.make_inputs(p, seed + 1, dtype, residual=residual, bias=bias)
    return d, p, a, b


def run_block(tvg, d, a, b, dtype, stride, relu_dw, relu_pw, hint=False, one_kernel=False):
    import torch
    dev = lambda v, t=dtype: to_dev(v, t)
    y = tvg.dwpw_fused(dev(a["x"]), dev(a["w"]), dev(a["scale"], "f32"), dev(a["shift"], "f32"),
                       dev(b["w"]), dev(b["scale"], "f32"), dev(b["shift"], "f32"),
                       dev(b["bias"], "f32"), dev(b["residual"]), stride=stride, relu_dw=relu_dw,
                       relu_pw=relu_pw, stream_out=hint, one_kernel=one_kernel)
    torch.cuda.synchronize()
    return y


def oracle_block(a, b, dtype, stride, relu_dw, relu_pw):
    return oracle.dwpw_fused(a["x"], a["w"], a["scale"], a["shift"], b["w"], b["scale"], b["shift"],
                             b["bias"], b["residual"], stride=stride, relu_dw=relu_dw,
                             relu_pw=relu_pw, store=dtype)


# (n, c, h, w, k): maps small enough for the one-kernel form (bf16, stride 1, c % 32 == 0)
BLOCK_FUSED = [(2, 256, 28, 28, 256), (2, 512, 14, 14, 512), (2, 1024, 7, 7, 1024),   # MobileNet
               (3, 64, 7, 7, 40), (1, 32, 6, 6, 8), (5, 96, 9, 5, 130), (2, 32, 28, 28, 64),
               (1, 64, 16, 8, 200), (7, 32, 5, 7, 64), (2, 128, 3, 40, 96), (1, 32, 33, 1, 70),
               (4, 160, 11, 13, 129), (1, 32, 8, 4, 1), (9, 64, 6, 6, 257), (1, 32, 56, 56, 64),
               (2, 64, 20, 62, 32)]


@pytest.mark.parametrize("cfg", BLOCK_FUSED, ids=lambda c: "x".join(map(str, c)))
def test_block_one_kernel_form(tvg, cfg):
    n, c, h, w, k = cfg
    seed = 7100 + sum(cfg)
    variant = seed % 4
    residual, bias = variant in (1, 3), variant in (2, 3)
    relu_dw, relu_pw = variant != 2, variant != 1
    d, p, a, b = block_inputs(n, c, h, w, k, 1, "bf16", seed, residual, bias)
    desc = tvg.ConvDesc(n, c, h, w, c, 3, 3, 1, 1, 1, 1, tvg.TVG_BF16, 0)
    assert tvg.tvg_dwpw_one_kernel(desc, k)
    want = oracle_block(a, b, "bf16", 1, relu_dw, relu_pw)
    y = run_block(tvg, d, a, b, "bf16", 1, relu_dw, relu_pw, one_kernel=True)
    assert tuple(y.shape) == p.y_shape()
    check(to_host(y), want, "bf16", tight=BLOCK_TIGHT)
    hinted = run_block(tvg, d, a, b, "bf16", 1, relu_dw, relu_pw, hint=True, one_kernel=True)
    import torch
    assert torch.equal(y.view(torch.int16), hinted.view(torch.int16))
    # the same problem as two kernels (a workspace is passed)
    two = run_block(tvg, d, a, b, "bf16", 1, relu_dw, relu_pw)
    check(to_host(two), want, "bf16", tight=BLOCK_TIGHT)


@pytest.mark.parametrize("cfg", [(2, 64, 14, 14, 64, 2, "bf16"), (1, 32, 112, 112, 64, 1, "bf16"),
                                 (1, 16, 9, 9, 8, 1, "f32"), (2, 24, 14, 14, 40, 1, "bf16"),
                                 (1, 8, 12, 16, 24, 2, "f32"), (2, 32, 5, 5, 16, 1, "bf16")],
                         ids=lambda c: "x".join(map(str, c)))
def test_block_two_kernel_form(tvg, cfg):
    n, c, h, w, k, stride, dtype = cfg
    d, p, a, b = block_inputs(n, c, h, w, k, stride, dtype, 7300 + sum(cfg[:6]), True, True)
    code = tvg.TVG_BF16 if dtype == "bf16" else tvg.TVG_F32
    desc = tvg.ConvDesc(n, c, h, w, c, 3, 3, stride, stride, 1, 1, code, 0)
    assert not tvg.tvg_dwpw_one_kernel(desc, k)
    y = run_block(tvg, d, a, b, dtype, stride, True, True)
    assert tuple(y.shape) == p.y_shape()
    check(to_host(y), oracle_block(a, b, dtype, stride, True, True), dtype,
          tight=BLOCK_TIGHT if dtype == "bf16" else None)


def test_block_one_kernel_form_batch32_full(tvg):
    """MobileNet's 14x14 block (512 -> 512) at batch 32, the benchmark's launch configuration:
    every output against the block oracle."""
    n, c, hw, k = 32, 512, 14, 512
    d, p, a, b = block_inputs(n, c, hw, hw, k, 1, "bf16", 7401, False, False)
    y = to_host(run_block(tvg, d, a, b, "bf16", 1, True, True, one_kernel=True))
    check(y, oracle_block(a, b, "bf16", 1, True, True), "bf16", tight=BLOCK_TIGHT)


@pytest.mark.parametrize("network", ["resnet18", "mobilenet"])
def test_body_in_a_planned_arena_matches_separate_tensors(tvg, network):
    """Every intermediate tensor of the chain placed by tvg_plan_arena in one arena (tensors that
    are never alive together share memory): the final output is bit-identical to the run with
    one allocation per tensor, twice in a row (the second run starts from a dirty arena)."""
    import torch
    steps = ti.resnet18_body(2) if network == "resnet18" else ti.mobilenet_body(2)
    config = 5 if network == "resnet18" else 6
    weights = body_weights(steps, config=config)
    images = ti.body_images(2, ti.layer_seed(config, 902))
    want = run_body_gpu(tvg, steps, images, weights)[steps[-1].dst]

    lives = ti.tensor_lives(steps)
    ids = [t for t in lives if t != 0]
    offsets, arena_bytes = tvg.tvg_plan_arena([lives[t] for t in ids])
    assert arena_bytes < sum(lives[t][0] for t in ids)
    arena = torch.full((arena_bytes,), 0x7F, dtype=torch.uint8, device="cuda")   # NaN patterns
    off = dict(zip(ids, offsets))
    dev_w = {k: {n: to_dev(v, "bf16" if n == "w" else "f32") for n, v in p.items()}
             for k, p in weights.items()}
    x0 = to_dev(images, "bf16")
    for rep in range(2):
        tensors = {0: x0}
        for st in steps:
            src = tensors[st.src]
            if st.op == "maxpool":
                n, c, h, w = src.shape
                shape = (n, c, (h - 1) // 2 + 1, (w - 1) // 2 + 1)
            else:
                shape = st.shape.y_shape()
            y = arena[off[st.dst]:off[st.dst] + lives[st.dst][0]].view(torch.bfloat16).view(shape)
            p = dev_w.get(st.layer_index)
            if st.op == "conv":
                res = None if st.residual is None else tensors[st.residual]
                tvg.conv2d_fused(src, p["w"], p["scale"], p["shift"], None, res, stride=st.shape.stride,
                                 pad=st.shape.pad, relu=st.relu, out=y)
            elif st.op == "dwconv":
                tvg.dwconv2d_fused(src, p["w"], p["scale"], p["shift"], None, None,
                                   stride=st.shape.stride, pad=1, relu=st.relu, out=y)
            else:
                tvg.maxpool2d_3x3s2(src, out=y)
            tensors[st.dst] = y
        torch.cuda.synchronize()
        got = tensors[steps[-1].dst]
        assert torch.equal(got.view(torch.int16), want.view(torch.int16)), rep
