"""The fp32 1x1 kernel (plan: fp32-small or generic, no knobs) against the oracle, every output: each instance
(pixels per lane, blocks, waves per reduction, chain length), channels and pixels that end inside a tile, maps of
odd size, strides, reductions shorter than the waves.  Bounds as for every single operator, and the
error of the sums against 64 bits."""
import numpy as np
import pytest

import oracle
import tvg_inputs as ti
from _util import check, dev_inputs, to_host

pytestmark = pytest.mark.gpu

# (n, ic, h, w, oc, stride), plan
EVERY_INSTANCE = [
    ((1, 32, 5, 5, 33, 1), (5, 32, 32)), ((2, 40, 7, 6, 40, 1), (5, 32, 32)), ((3, 56, 6, 6, 31, 2), (5, 32, 32)),
    ((40, 32, 10, 11, 70, 1), (5, 32, 64)), ((40, 64, 11, 9, 70, 1), (5, 32, 64)), ((80, 48, 9, 9, 96, 1), (5, 32, 128)),
    ((80, 40, 10, 9, 96, 1), (5, 32, 128)), ((20, 264, 14, 12, 96, 1), (5, 32, 64)), ((50, 72, 12, 12, 97, 1), (5, 32, 128)),
    ((8, 72, 31, 28, 121, 1), (0, 64, 64)), ((64, 72, 31, 14, 121, 1), (0, 64, 128)), ((8, 64, 55, 57, 126, 1), (0, 64, 64)),
    ((8, 128, 28, 28, 256, 1), (0, 64, 64)), ((40, 256, 5, 63, 50, 1), (0, 64, 64)), ((128, 256, 1, 77, 256, 1), (0, 64, 128)),
    ((16, 64, 57, 57, 128, 2), (0, 64, 64)), ((17, 256, 29, 30, 128, 2), (5, 32, 64)), ((33, 136, 33, 31, 128, 1), (0, 64, 64)),
    ((22, 264, 42, 33, 192, 1), (0, 64, 128)), ((22, 264, 41, 33, 192, 1), (0, 64, 128)), ((22, 264, 44, 33, 192, 1), (0, 64, 128)),
]


# Strides from 3 on and long rows, narrow tiles in place of the gather kernel's; two totals and four; 64-pixel tiles of
# single pixels; chains of 16 in 128-pixel tiles.
EVERY_INSTANCE += [
    ((1, 512, 14, 14, 512, 3), (0, 32, 32)), ((7, 152, 29, 31, 70, 4), (0, 32, 32)), ((3, 40, 26, 97, 33, 3), (0, 32, 32)),
    ((2, 96, 1, 2050, 90, 1), (0, 32, 64)), ((41, 72, 40, 50, 125, 3), (0, 32, 128)), ((40, 32, 50, 50, 70, 3), (0, 32, 128)),
    ((8, 128, 57, 57, 120, 2), (0, 64, 64)), ((1, 1032, 5, 5, 40, 1), (5, 32, 32)), ((9, 1048, 7, 9, 70, 2), (5, 32, 32)),
    ((30, 128, 56, 49, 128, 1), (0, 64, 128)),
]


@pytest.mark.parametrize("tail", ["plain", "bias+residual"])
@pytest.mark.parametrize("cfg,plan", EVERY_INSTANCE, ids=lambda c: "x".join(map(str, c)))
def test_f32_1x1_every_instance(tvg, cfg, plan, tail):
    n, ic, h, w, oc, stride = cfg
    desc = tvg.ConvDesc(n, ic, h, w, oc, 1, 1, stride, stride, 0, 0, tvg.TVG_F32, 0)
    assert tvg.tvg_conv2d_get_plan(desc) == plan and not any(tvg.tvg_conv2d_get_knobs(desc))
    assert tvg.tvg_conv2d_workspace_size(desc) == 0
    full = tail != "plain"
    inp = ti.make_inputs(ti.ConvShape("pw", n, ic, h, w, oc, 1, 1, stride, 0), 8700 + sum(cfg), "f32", residual=full, bias=full)
    d = dev_inputs(inp, "f32")
    y = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], d["bias"], d["residual"], stride=stride, relu=full)
    want = oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"], inp["residual"],
                               stride=(stride,) * 2, pad=(0, 0), relu=full)
    check(to_host(y), want, "f32", cfg)


# One rounding of a partial sum is 2.5e-8 rms of it, and a chain of m products errs by about 2.5e-8 sqrt(m / 2) of its
# sum; chains of 8 (16, 32) channels added up one after the other give below 1.1e-7 for these, one chain of all 1.8e-7
# to 5.7e-7.
@pytest.mark.parametrize("cfg", [(1, 512, 14, 14, 512, 1), (4, 256, 14, 14, 512, 1), (8, 256, 28, 28, 256, 1), (3, 1000, 26, 26, 228, 1)],
                         ids=lambda c: "x".join(map(str, c)))
def test_f32_1x1_sums_in_short_chains(tvg, cfg):
    import torch
    n, ic, h, w, oc, _ = cfg
    inp = ti.make_inputs(ti.ConvShape("sums", n, ic, h, w, oc, 1, 1, 1, 0), 8800 + sum(cfg), "f32")
    one, none = torch.ones(oc), torch.zeros(oc)
    got = tvg.conv2d_fused(torch.from_numpy(inp["x"]).cuda(), torch.from_numpy(inp["w"]).cuda(), one.cuda(), none.cuda(), relu=False)
    want = np.matmul(inp["w"].astype(np.float64).reshape(oc, ic), inp["x"].astype(np.float64).reshape(n, ic, h * w))
    err = np.linalg.norm(got.cpu().numpy().astype(np.float64).reshape(n, oc, h * w) - want) / np.linalg.norm(want)
    assert err <= 1.3e-7, (cfg, err)


# The same under a stride (16 channels per chain up to 511: 7.1e-8 of a chain, 5e-8 of eight of them added up, 9.2e-8 with
# the last sums; 32 per chain 1.1e-7) and for long reductions of few tiles (64 chains of 8 per wave: in four totals
# 5e-8, 7.1e-8 and four levels of sums, 1.0e-7; in two totals 1.2e-7).  The kernels that ran these before: 0.98e-7, 1.22e-7.
@pytest.mark.parametrize("cfg,bound", [((32, 256, 28, 28, 256, 2), 1.05e-7), ((64, 264, 14, 14, 512, 2), 1.05e-7), ((1, 2048, 7, 7, 512, 1), 1.2e-7)],
                         ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else "")
def test_f32_1x1_sums_of_strided_and_long_reductions(tvg, cfg, bound):
    import torch
    n, ic, h, w, oc, stride = cfg
    g = torch.Generator().manual_seed(8850 + sum(cfg))
    x, wt = torch.rand((n, ic, h, w), generator=g) * 2 - 1, torch.randn((oc, ic, 1, 1), generator=g) * (2.0 / ic) ** 0.5
    got = tvg.conv2d_fused(x.cuda(), wt.cuda(), torch.ones(oc).cuda(), torch.zeros(oc).cuda(), stride=stride, relu=False)
    want = torch.matmul(wt.double().view(oc, ic), x[:, :, ::stride, ::stride].double().reshape(n, ic, -1))
    err = float((got.cpu().double().view(want.shape) - want).norm() / want.norm())
    assert err <= bound, (cfg, err)


@pytest.mark.parametrize("shape", [(2, 64, 8, 8, 40), (1, 512, 14, 14, 512)])
def test_f32_1x1_unaligned_pointers(tvg, shape):
    """x, y and the residual at any element, without a workspace as queried."""
    import torch
    n, ic, h, w, oc = shape
    inp = ti.make_inputs(ti.ConvShape("pwa", n, ic, h, w, oc, 1, 1, 1, 0), 8900, "f32", residual=True)
    d = dev_inputs(inp, "f32")
    want = oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], None, inp["residual"], stride=(1, 1), pad=(0, 0), relu=True)
    def at(t, off):
        store = torch.zeros(t.numel() + 8, device="cuda")
        v = store[off:off + t.numel()].view(t.shape)
        v.copy_(t)
        return v
    desc = tvg.ConvDesc(n, ic, h, w, oc, 1, 1, 1, 1, 0, 0, tvg.TVG_F32, tvg.TVG_RELU)
    for ox, oy in ((0, 1), (1, 0)):
        y = at(torch.zeros_like(d["residual"]), oy)
        rc = tvg.tvg_conv2d_fused(desc, at(d["x"], ox), d["w"], d["scale"], d["shift"], None, at(d["residual"], oy), y, None, 0, None)
        assert rc == 0, tvg.status_string(rc)
        check(to_host(y), want, "f32", (shape, ox, oy))


@pytest.mark.parametrize("cfg", [(1, 512, 14, 14, 512, 1), (3, 56, 6, 6, 31, 2), (8, 128, 28, 28, 256, 1)], ids=lambda c: "x".join(map(str, c)))
def test_f32_1x1_nan_stays_in_its_pixel(tvg, cfg):
    """A NaN in the input comes out as one without a ReLU, in every channel of its pixel and nowhere else."""
    import torch
    n, ic, h, w, oc, stride = cfg
    d = dev_inputs(ti.make_inputs(ti.ConvShape("nan", n, ic, h, w, oc, 1, 1, stride, 0), 8950, "f32"), "f32")
    clean = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], stride=stride, relu=False)
    d["x"][n - 1, ic - 1, 2 * stride, stride] = float("nan")
    y = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], stride=stride, relu=False)
    assert bool(torch.isnan(y[n - 1, :, 2, 1]).all())
    y[n - 1, :, 2, 1] = clean[n - 1, :, 2, 1]
    assert torch.equal(y, clean)


@pytest.mark.parametrize("cfg", [(1, 512, 14, 14, 512, 1), (1, 1024, 7, 7, 200, 1), (3, 56, 6, 6, 31, 2), (8, 128, 28, 28, 256, 1), (1, 512, 14, 14, 128, 3)],
                         ids=lambda c: "x".join(map(str, c)))
def test_f32_1x1_weights_in_a_parameter_buffer(tvg, cfg):
    """Weights and x that begin at any element of a larger buffer have the bits of aligned ones: no other kernel, whose
    sums come in another order, takes their place."""
    import torch
    n, ic, h, w, oc, stride = cfg
    d = dev_inputs(ti.make_inputs(ti.ConvShape("flat", n, ic, h, w, oc, 1, 1, stride, 0), 8970, "f32"), "f32")
    want = tvg.conv2d_fused(d["x"], d["w"], d["scale"], d["shift"], stride=stride, relu=False)
    def at(t, off):
        store = torch.full((t.numel() + 8,), float("nan"), device="cuda")
        v = store[off:off + t.numel()].view(t.shape)
        v.copy_(t)
        return v
    for ox, ow in ((0, 1), (0, 2), (3, 3), (1, 0)):
        y = tvg.conv2d_fused(at(d["x"], ox), at(d["w"], ow), d["scale"], d["shift"], stride=stride, relu=False)
        assert torch.equal(y, want), (ox, ow)
