"""A NaN in x comes out as a NaN, not as minus infinity, where no ReLU is asked for: in every output whose window holds it
and in no other, for every kernel and both tails (wide and element-wise)."""
import pytest

import tvg_inputs as ti
from _util import dev_inputs

pytestmark = pytest.mark.gpu

# dtype, (n, ic, h, w, oc, filter, stride), kernel and output channels per tile of the plan
DENSE = [
    ("bf16", (2, 128, 28, 28, 72, 3, 1), (1, 16)), ("bf16", (2, 96, 13, 11, 33, 1, 1), (4, 16)), ("bf16", (3, 256, 14, 14, 40, 3, 2), (1, 16)),
    ("bf16", (32, 512, 14, 14, 128, 1, 1), (4, 64)), ("bf16", (64, 512, 7, 7, 512, 1, 1), (4, 64)), ("bf16", (40, 64, 28, 28, 128, 1, 2), (4, 64)),
    ("bf16", (16, 64, 56, 56, 64, 3, 1), (1, 64)), ("bf16", (64, 128, 28, 28, 128, 3, 1), (7, 64)), ("bf16", (64, 512, 7, 7, 512, 3, 1), (7, 64)),
    # strips in windows, under a stride, and with four groups of waves
    ("bf16", (24, 192, 56, 56, 64, 3, 1), (7, 64)), ("bf16", (64, 256, 14, 14, 512, 3, 2), (7, 64)), ("bf16", (64, 256, 14, 14, 64, 3, 1), (7, None)),
    ("bf16", (4, 3, 64, 64, 64, 7, 2), (3, 64)), ("bf16", (2, 45, 23, 21, 40, 3, 1), (0, None)),
    ("f32", (1, 64, 28, 28, 64, 3, 1), (5, None)), ("f32", (1, 3, 64, 64, 40, 7, 2), (5, None)), ("f32", (32, 64, 28, 28, 64, 3, 1), (0, 64)),
    ("f32", (1, 512, 14, 14, 96, 1, 1), (5, 32)), ("f32", (2, 45, 23, 21, 40, 3, 1), (0, None)),
]
# ... of the two other 3x3 kernels, which a caller names by their stages
NAMED = [("bf16", (64, 128, 28, 28, 128, 3, 1), (2, 64)), ("bf16", (64, 512, 7, 7, 512, 3, 1), (2, 64)), ("bf16", (64, 256, 14, 14, 512, 3, 2), (2, 64)),
         ("bf16", (8, 64, 56, 56, 64, 3, 1), (1, 64))]
DEPTHWISE = [(dtype, c, h, w, stride) for dtype in ("f32", "bf16")
             for c, h, w, stride in ((64, 28, 28, 1), (32, 56, 56, 2), (40, 7, 7, 1), (16, 13, 11, 2), (8, 112, 112, 1), (24, 19, 33, 1))]


def check_nan(call, x, at, r, stride, channel=None):
    """call(x) without a ReLU, clean and with a NaN at [image, channel, row, column]."""
    import torch
    clean = call(x)
    x[at] = float("nan")
    y = call(x)
    hit = torch.zeros(y.shape, dtype=torch.bool, device=y.device)
    rows = [o for o in range(y.shape[2]) if abs(o * stride - at[2]) <= r // 2]
    cols = [o for o in range(y.shape[3]) if abs(o * stride - at[3]) <= r // 2]
    assert rows and cols
    hit[at[0], slice(None) if channel is None else channel, rows[0]:rows[-1] + 1, cols[0]:cols[-1] + 1] = True
    assert bool(torch.isnan(y[hit]).all())
    assert torch.equal(y[~hit], clean[~hit])


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("dtype,cfg,plan", DENSE, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else c)
def test_nan_stays_one(tvg, dtype, cfg, plan, residual):
    n, ic, h, w, oc, r, stride = cfg
    desc = tvg.ConvDesc(n, ic, h, w, oc, r, r, stride, stride, r // 2, r // 2, tvg.TVG_BF16 if dtype == "bf16" else tvg.TVG_F32, 0)
    got = tvg.tvg_conv2d_get_plan(desc)
    assert got[0] == plan[0] and plan[1] in (None, got[1])
    d = dev_inputs(ti.make_inputs(ti.ConvShape("nan", n, ic, h, w, oc, r, r, stride, r // 2), 9700 + sum(cfg), dtype, residual=residual), dtype)
    check_nan(lambda x: tvg.conv2d_fused(x, d["w"], d["scale"], d["shift"], None, d["residual"], stride=stride, pad=r // 2, relu=False),
              d["x"], (n - 1, ic - 1, 2 * stride, h - 1 - (h - 1) % stride if w == h else 2 * stride), r, stride)


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("dtype,cfg,plan", NAMED, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else c)
def test_nan_stays_one_in_a_named_kernel(tvg, dtype, cfg, plan, residual):
    n, ic, h, w, oc, r, stride = cfg
    desc = tvg.ConvDesc(n, ic, h, w, oc, r, r, stride, stride, 1, 1, tvg.TVG_BF16, 0)
    assert tvg.tvg_conv2d_set_knobs(desc, (0, 0, plan[0], 0, 0, 0)) == 0
    try:
        test_nan_stays_one(tvg, dtype, cfg, plan, residual)
    finally:
        tvg.tvg_conv2d_set_knobs(desc, None)


@pytest.mark.parametrize("dtype,c,h,w,stride", DEPTHWISE)
def test_nan_stays_one_depthwise(tvg, dtype, c, h, w, stride):
    d = dev_inputs(ti.make_inputs(ti.ConvShape("nan", 2, c, h, w, c, 3, 3, stride, 1, depthwise=True), 9800 + c + h, dtype), dtype)
    check_nan(lambda x: tvg.dwconv2d_fused(x, d["w"], d["scale"], d["shift"], stride=stride, pad=1, relu=False),
              d["x"], (1, c - 1, 2 * stride, 2 * stride), 3, stride, c - 1)


@pytest.mark.parametrize("one_kernel", [False, True])
def test_nan_stays_one_in_a_block(tvg, one_kernel):
    import torch
    g = torch.Generator(device="cuda").manual_seed(9900)
    rand = lambda *s: torch.rand(s, generator=g, device="cuda") * 2 - 1
    x, wd, wp = rand(2, 64, 14, 14).bfloat16(), rand(64, 1, 3, 3).bfloat16(), rand(128, 64, 1, 1).bfloat16()
    one = lambda k: (torch.ones(k, device="cuda"), torch.zeros(k, device="cuda"))
    check_nan(lambda x: tvg.dwpw_fused(x, wd, *one(64), wp, *one(128), relu_dw=False, relu_pw=False, one_kernel=one_kernel),
              x, (1, 63, 2, 2), 3, 1)
