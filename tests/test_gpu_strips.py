"""The bf16 3x3 kernel of strips (knobs stages = 1, row_loads = 2; by rule it stands in for the kernels that are reported)
against the oracle, every output: strips of 4 to 8 rows, rows of one to four strips of an even and an odd number of pixels
and rows cut into windows, both strides, one, two and four groups of waves, the last strip and the last tile partly outside,
channels that end inside a tile, reductions of one to twenty chunks, several tiles per workgroup.  Bounds as for every single operator."""
import pytest

import oracle
import tvg_inputs as ti
from _util import check, dev_inputs, to_host

pytestmark = pytest.mark.gpu

# (n, ic, h, w, oc), rows of a strip that planning picks there (groups: 1, for odd rows 2, and 4)
SHAPES = [
    ((2, 64, 9, 6, 70), 4), ((3, 160, 14, 14, 130), 4), ((1, 96, 13, 18, 40), 4), ((2, 128, 28, 28, 72), 4), ((1, 32, 5, 32, 33), 4), ((1, 512, 3, 8, 17), 4),
    ((70, 64, 3, 2, 16), 4), ((1, 32, 1, 1, 1), 4), ((3, 128, 7, 7, 130), 4), ((2, 64, 13, 13, 80), 4), ((1, 192, 17, 21, 64), 4), ((2, 64, 9, 31, 20), 4),
    ((130, 64, 5, 26, 16), 5), ((260, 64, 5, 14, 16), 5), ((520, 64, 5, 5, 16), 5), ((130, 64, 5, 19, 16), 5),
    ((130, 64, 6, 20, 16), 6), ((520, 64, 6, 6, 40), 6), ((260, 64, 6, 13, 16), 6), ((130, 64, 6, 29, 16), 6),
    ((130, 64, 7, 28, 20), 7), ((260, 32, 7, 14, 16), 7), ((520, 64, 7, 7, 16), 7), ((130, 64, 7, 25, 16), 7),
    ((390, 64, 8, 30, 16), 8), ((1560, 64, 8, 8, 16), 8), ((780, 64, 8, 16, 16), 8), ((780, 64, 8, 15, 16), 8), ((1560, 64, 8, 3, 16), 8),
    # windows: rows of 36 to 112 pixels
    ((1, 64, 5, 36, 16), 4), ((2, 96, 13, 56, 70), 4), ((1, 32, 9, 112, 20), 4), ((70, 64, 5, 36, 16), 5), ((70, 64, 16, 36, 16), 6), ((70, 64, 7, 40, 16), 7), ((140, 64, 8, 60, 16), 8),
    # reductions that four groups split too, even and odd rows, windows
    ((33, 256, 5, 14, 40), 4), ((2, 384, 9, 31, 33), 4), ((5, 128, 2, 5, 64), 4), ((1, 640, 6, 26, 97), 4), ((1, 128, 9, 112, 20), 4),
    # two and three tiles per workgroup, of one and of several channel tiles, pixel tiles first and (many images) channel tiles first
    ((1100, 64, 7, 28, 16), 7), ((300, 32, 14, 14, 200), 7), ((700, 96, 8, 10, 130), 8), ((260, 64, 7, 28, 130), 7),
    # more tiles than workgroups that walk: odd rows and split reductions, which have a workgroup per tile
    ((1100, 64, 7, 9, 16), 7), ((560, 128, 4, 28, 40), 4), ((560, 128, 4, 27, 40), 4),
]

# ... under a stride of 2
STRIDE2 = [
    ((1, 64, 5, 6, 16), 4), ((3, 160, 14, 14, 130), 4), ((1, 96, 13, 18, 40), 4), ((2, 128, 28, 28, 72), 4), ((1, 512, 3, 8, 17), 4), ((1, 32, 1, 1, 1), 4),
    ((70, 64, 3, 2, 16), 4), ((1, 64, 9, 3, 33), 4), ((3, 128, 7, 7, 130), 4), ((2, 64, 13, 13, 80), 4), ((1, 192, 17, 21, 64), 4), ((2, 64, 9, 31, 20), 4), ((1, 64, 6, 32, 24), 4),
    ((1, 64, 5, 40, 16), 4), ((2, 96, 14, 56, 70), 4), ((1, 32, 9, 112, 20), 4), ((1, 64, 6, 36, 16), 4),
    ((260, 64, 9, 14, 16), 5), ((130, 64, 9, 21, 16), 5), ((70, 64, 9, 40, 16), 5), ((130, 64, 11, 26, 16), 6), ((520, 64, 11, 3, 16), 6),
    ((520, 64, 13, 6, 16), 7), ((130, 64, 13, 28, 40), 7), ((260, 64, 13, 13, 16), 7), ((70, 64, 13, 40, 16), 7), ((300, 32, 28, 28, 100), 7), ((300, 64, 13, 13, 130), 7), ((1100, 64, 13, 11, 16), 7),
]


def tile_pixels(cfg, b, stride):
    """Up to four strips of b rows x 8 input pixels: side by side in a row, or in part of a long one, and rows of strips."""
    n, _, h, w, _ = cfg
    side = min(-(-w // 8), 4)
    windows = 1 if w <= 32 else -(-(w - 8) // 24) if stride == 1 else -(-(-(-w // 8) - 1) // 3)
    rows = min(4 // side, n * windows * -(-(-(-h // stride)) // b))
    return rows * side * b * 8 // stride


def _check(tvg, cfg, b, kg, residual, bias, relu, stride=1):
    n, ic, h, w, oc = cfg
    desc = tvg.ConvDesc(n, ic, h, w, oc, 3, 3, stride, stride, 1, 1, tvg.TVG_BF16, 0)
    inp = ti.make_inputs(ti.ConvShape("strips", n, ic, h, w, oc, 3, 3, stride, 1), 10300 + sum(cfg), "bf16", residual=residual, bias=bias)
    d = dev_inputs(inp, "bf16")
    want = oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"] if bias else None,
                               inp["residual"] if residual else None, stride=(stride, stride), pad=(1, 1), relu=relu)
    assert tvg.tvg_conv2d_set_knobs(desc, (0, 0, 1, kg, 0, 2)) == 0
    try:
        assert tvg.tvg_conv2d_get_plan(desc) == (7, 32 if kg == 4 else 64, tile_pixels(cfg, b, stride)) and tvg.tvg_conv2d_get_knobs(desc) == (0, 0, 1, kg, 0, 2)
        ys = [tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], d["bias"] if bias else None, d["residual"] if residual else None,
                               stride=stride, pad=1, relu=relu, stream_out=hint) for hint in (False, True)]
    finally:
        tvg.tvg_conv2d_set_knobs(desc, None)
    assert ys[0].view(-1).equal(ys[1].view(-1))                        # the store hint changes no bits, nor does a repetition
    check(to_host(ys[0]), want, "bf16", (cfg, b, kg))


# two groups: odd rows; four: strips of four rows; both: a multiple of their number of chunks
GROUPED = [(cfg, b, kg) for kg in (1, 2, 4) for cfg, b in SHAPES
           if not (kg == 2 and (cfg[3] % 2 == 0 or cfg[1] % 64 != 0)) and not (kg == 4 and (b != 4 or cfg[1] % 128 != 0))]


@pytest.mark.parametrize("tail", ["plain", "bias+residual"])
@pytest.mark.parametrize("cfg,b,kg", GROUPED, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_strips_every_instance(tvg, cfg, b, kg, tail):
    full = tail != "plain"
    _check(tvg, cfg, b, kg, full, full, full)


@pytest.mark.parametrize("tail", ["plain", "bias+residual"])
@pytest.mark.parametrize("cfg,b", STRIDE2, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_strips_every_instance_stride_2(tvg, cfg, b, tail):
    full = tail != "plain"
    _check(tvg, cfg, b, 1, full, full, full, 2)


def at(t, off):
    """A copy of t that starts `off` elements into a buffer of zeros, and that buffer."""
    import torch
    buf = torch.zeros(t.numel() + 24, dtype=torch.bfloat16, device="cuda")
    v = buf[off:off + t.numel()].view(t.shape)
    v.copy_(t)
    return v, buf


@pytest.mark.parametrize("cfg", [(3, 128, 28, 28, 64), (5, 128, 7, 7, 128)], ids=lambda c: "x".join(map(str, c)))
def test_strips_unaligned_pixels_get_the_kernel_behind(tvg, cfg):
    """x off a 16-byte address: another kernel, the same result up to the order of the sums."""
    import torch
    n, ic, h, w, oc = cfg
    desc = tvg.ConvDesc(n, ic, h, w, oc, 3, 3, 1, 1, 1, 1, tvg.TVG_BF16, 0)
    inp = ti.make_inputs(ti.ConvShape("strips", n, ic, h, w, oc, 3, 3, 1, 1), 10500, "bf16", residual=True)
    d = dev_inputs(inp, "bf16")
    want = oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], None, inp["residual"], stride=(1, 1), pad=(1, 1), relu=False)
    assert tvg.tvg_conv2d_set_knobs(desc, (0, 0, 1, 0, 0, 2)) == 0
    try:
        for ox in (0, 2):
            y = torch.zeros_like(d["residual"])
            rc = tvg.tvg_conv2d_fused(desc, at(d["x"], ox)[0], d["w"], d["scale"], d["shift"], None, d["residual"], y, None, 0, None)
            assert rc == 0, tvg.status_string(rc)
            check(to_host(y), want, "bf16", ox)
    finally:
        tvg.tvg_conv2d_set_knobs(desc, None)


# n, ic, h, w, oc, stride, groups: rows that end in 8, 4, 2 and an odd number of pixels, windows, both strides, split reductions
ANY_ELEMENT = [(3, 128, 28, 28, 64, 1, 1), (2, 64, 9, 30, 20, 1, 1), (2, 64, 8, 16, 33, 1, 1), (5, 128, 7, 7, 128, 1, 2), (2, 96, 13, 56, 70, 1, 1), (1, 64, 9, 36, 20, 1, 1),
               (2, 128, 14, 14, 40, 1, 4), (2, 64, 13, 15, 16, 1, 1), (2, 64, 28, 28, 64, 2, 1), (2, 64, 14, 14, 70, 2, 1), (3, 64, 13, 13, 20, 2, 1), (2, 64, 14, 56, 24, 2, 1)]


@pytest.mark.parametrize("cfg", ANY_ELEMENT, ids=lambda c: "x".join(map(str, c)))
def test_strips_outputs_at_any_element(tvg, cfg):
    """y and the residual at any element: the bits of an aligned call, and nothing written outside y."""
    import torch
    n, ic, h, w, oc, stride, kg = cfg
    desc = tvg.ConvDesc(n, ic, h, w, oc, 3, 3, stride, stride, 1, 1, tvg.TVG_BF16, 0)
    d = dev_inputs(ti.make_inputs(ti.ConvShape("strips", n, ic, h, w, oc, 3, 3, stride, 1), 10550 + sum(cfg), "bf16", residual=True), "bf16")
    assert tvg.tvg_conv2d_set_knobs(desc, (0, 0, 1, kg, 0, 2)) == 0
    try:
        assert tvg.tvg_conv2d_get_plan(desc)[0] == 7
        want = None
        for oy, orr in ((0, 0), (1, 0), (2, 0), (4, 0), (0, 1), (0, 2), (0, 4), (3, 5), (2, 6)):
            y, buf = at(torch.full_like(d["residual"], float("nan")), oy)
            rc = tvg.tvg_conv2d_fused(desc, d["x"], d["w"], d["scale"], d["shift"], None, at(d["residual"], orr)[0], y, None, 0, None)
            assert rc == 0, tvg.status_string(rc)
            want = y.clone() if want is None else want
            assert torch.equal(y, want), (oy, orr)
            assert not bool(buf[:oy].any()) and not bool(buf[oy + y.numel():].any()), (oy, orr)
        # in place: y may be the residual
        v, _ = at(d["residual"], 1)
        assert tvg.tvg_conv2d_fused(desc, d["x"], d["w"], d["scale"], d["shift"], None, v, v, None, 0, None) == 0
        assert torch.equal(v, want)
    finally:
        tvg.tvg_conv2d_set_knobs(desc, None)


# n, ic, h, w, channels of the two heads, stride
@pytest.mark.parametrize("cfg", [(32, 128, 28, 28, 128, 64, 1), (64, 256, 14, 14, 64, 256, 1), (64, 128, 16, 16, 128, 40, 1), (128, 256, 14, 14, 512, 512, 2),
                                 (24, 192, 56, 56, 64, 40, 1)], ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("centre", [True, False])
def test_two_heads_have_the_bits_of_separate_calls_in_strips(tvg, cfg, centre):
    import torch
    n, ic, h, w, k1, k2, stride = cfg
    r2 = 1 if centre else 3
    plan = lambda k, r: tvg.tvg_conv2d_get_plan(tvg.ConvDesc(n, ic, h, w, k, r, r, stride, stride, r // 2, r // 2, tvg.TVG_BF16, 0))
    assert plan(k1, 3)[0] == 7 and plan(k2, r2)[0] == (4 if centre else 7)
    g = torch.Generator(device="cuda").manual_seed(10600 + sum(cfg))
    def rand(*shape):
        return torch.rand(shape, generator=g, device="cuda") * 2 - 1
    x, w1, w2 = (rand(*s).to(torch.bfloat16) for s in ((n, ic, h, w), (k1, ic, 3, 3), (k2, ic, r2, r2)))
    scale, shift = rand(k1 + k2), rand(k1 + k2)
    joined = torch.zeros(k1 + k2, ic, 3, 3, dtype=torch.bfloat16, device="cuda")
    joined[:k1] = w1
    if centre:
        joined[k1:, :, 1, 1] = w2[:, :, 0, 0]
    else:
        joined[k1:] = w2
    want1 = tvg.conv2d_fused(x, w1, scale[:k1], shift[:k1], stride=stride, pad=1, relu=True)
    want2 = tvg.conv2d_fused(x, w2, scale[k1:].clone(), shift[k1:].clone(), stride=stride, pad=r2 // 2, relu=False)
    y1, y2 = torch.full_like(want1, float("nan")), torch.full_like(want2, float("nan"))
    desc = tvg.ConvDesc(n, ic, h, w, k1 + k2, 3, 3, stride, stride, 1, 1, tvg.TVG_BF16, tvg.TVG_RELU)
    rc = tvg.tvg_conv2d_fused_dual(desc, k1, tvg.TVG_CENTRE_TAP_ONLY if centre else 0, x, joined, scale, shift, None, None, y1, y2)
    assert rc == 0, tvg.status_string(rc)
    assert torch.equal(y1, want1) and torch.equal(y2, want2)


# rows, columns, stride, groups of waves
@pytest.mark.parametrize("h,w,stride,kg", [(14, 14, 1, 1), (28, 28, 1, 1), (7, 7, 1, 1), (9, 18, 1, 1), (6, 56, 1, 1), (7, 7, 1, 2), (13, 13, 1, 2), (9, 31, 1, 2),
                                           (14, 14, 1, 4), (7, 7, 1, 4), (9, 18, 1, 4), (6, 56, 1, 4), (14, 14, 2, 1), (28, 28, 2, 1), (7, 7, 2, 1), (9, 18, 2, 1),
                                           (13, 31, 2, 1), (6, 56, 2, 1)])
def test_strips_infinity_stays_in_its_window(tvg, h, w, stride, kg):
    """Pixels at the end of a row and of a strip, whose neighbours in LDS belong to other rows and images, and the first channel
    of every group's share of the reduction."""
    import torch
    desc = tvg.ConvDesc(3, 128, h, w, 64, 3, 3, stride, stride, 1, 1, tvg.TVG_BF16, 0)
    d = dev_inputs(ti.make_inputs(ti.ConvShape("strips", 3, 128, h, w, 64, 3, 3, stride, 1), 10700, "bf16"), "bf16")
    assert tvg.tvg_conv2d_set_knobs(desc, (0, 0, 1, kg, 0, 2)) == 0
    try:
        assert tvg.tvg_conv2d_get_plan(desc)[0] == 7 and tvg.tvg_conv2d_get_knobs(desc)[3] == kg
        call = lambda x: tvg.conv2d_fused(x, d["w"], d["scale"], d["shift"], stride=stride, pad=1, relu=False)
        clean = call(d["x"])
        for i, (row, col) in enumerate(((3, w - 1), (4, 0), (h - 1, w - 1), (0, 0), (2, w // 2), (2, w // 2 - 1))):
            x = d["x"].clone()
            x[1, 32 * i % 128, row, col] = float("inf")
            y = call(x)
            hit = torch.zeros_like(y, dtype=torch.bool)
            rows = [o for o in range(y.shape[2]) if abs(o * stride - row) <= 1]
            cols = [o for o in range(y.shape[3]) if abs(o * stride - col) <= 1]
            if rows and cols:
                hit[1, :, rows[0]:rows[-1] + 1, cols[0]:cols[-1] + 1] = True
            assert not bool(torch.isfinite(y[hit]).any()) and torch.equal(y[~hit], clean[~hit]), (row, col)
    finally:
        tvg.tvg_conv2d_set_knobs(desc, None)
