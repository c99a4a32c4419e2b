"""What a call does with less scratch than the size query reports (include/tvg.h): bf16 problems whose
weights are packed first run on the generic kernel while its partial sums fit, everything else is an error."""
import pytest

import oracle
import tvg_inputs as ti
import paper_1802_04799_amd as pkg
from _util import BLOCK_TIGHT, check, dev_inputs, to_host

BF16 = pkg.TVG_BF16
FAKE = 0x10000          # a 256-byte aligned "device pointer" for calls that must fail before touching it
ARGS = (FAKE, FAKE, FAKE, FAKE, None, None, FAKE)


def generic_workspace(desc):
    """The generic kernel's workspace for this problem (its tile fixed to the one its own rule takes)."""
    assert pkg.tvg_conv2d_set_tile(desc, 128 if desc.k > 64 else 64, 128) == 0
    try:
        return pkg.tvg_conv2d_workspace_size(desc)
    finally:
        pkg.tvg_conv2d_set_tile(desc, 0, 0)


def test_too_little_for_either_kernel_is_an_error():
    d = pkg.ConvDesc(1, 509, 7, 7, 512, 3, 3, 1, 1, 1, 1, BF16, 0)
    need, least = pkg.tvg_conv2d_workspace_size(d), generic_workspace(d)
    assert 0 < least < need
    assert pkg.tvg_conv2d_fused(d, *ARGS, None, 0, 0) == 4
    assert pkg.tvg_conv2d_fused(d, *ARGS, FAKE, least - 1, 0) == 4
    assert pkg.tvg_conv2d_fused(d, *ARGS, FAKE + 64, need, 0) == 4
    big = pkg.ConvDesc(1, 4100, 14, 14, 1028, 3, 3, 1, 1, 1, 1, BF16, 0)
    assert min(pkg.tvg_conv2d_workspace_size(big), generic_workspace(big)) > pkg.tvg_static_scratch_bytes()
    assert pkg.tvg_conv2d_fused_static(big, *ARGS, 0) == 4


def block(n, c, hw, k):
    """(descriptor, bytes of t, the generic kernel's workspace for the 1x1 stage)"""
    dw = pkg.ConvDesc(n, c, hw, hw, c, 3, 3, 1, 1, 1, 1, BF16, pkg.TVG_RELU)
    pw = pkg.ConvDesc(n, c, hw, hw, k, 1, 1, 1, 1, 0, 0, BF16, 0)
    return dw, (n * c * hw * hw * 2 + 255) // 256 * 256, generic_workspace(pw)


def test_a_block_without_room_for_the_partial_sums_is_an_error():
    dw, t, least = block(1, 1021, 5, 300)
    assert least > 0 and pkg.tvg_dwpw_workspace_size(dw, 300) > t + least
    args = [FAKE] * 7 + [None, None, FAKE]
    assert pkg.tvg_dwpw_fused(dw, 300, 0, *args, FAKE, t + least - 1, 0) == 4
    assert pkg.tvg_dwpw_fused(dw, 300, 0, *args, FAKE + 64, t + least, 0) == 4


def _run(tvg, sh, workspace_bytes, offset=0, static=False):
    """y of the problem with a workspace of that many bytes (None: NULL) at that offset."""
    import torch
    inp = ti.make_inputs(sh, 6500, "bf16", residual=True, bias=True)
    d = dev_inputs(inp, "bf16")
    desc = tvg.ConvDesc(sh.n, sh.ic, sh.h, sh.w, sh.oc, sh.r, sh.s, sh.stride, sh.stride, sh.pad, sh.pad, BF16, tvg.TVG_RELU)
    y = torch.full(sh.y_shape(), float("nan"), dtype=torch.bfloat16, device="cuda")
    tensors = (d["x"], d["w"], d["scale"], d["shift"], d["bias"], d["residual"], y)
    if static:
        assert tvg.tvg_conv2d_fused_static(desc, *tensors) == 0
    else:
        ws = None if workspace_bytes is None else torch.empty(workspace_bytes + offset, dtype=torch.uint8, device="cuda")[offset:]
        assert tvg.tvg_conv2d_fused(desc, *tensors, ws, workspace_bytes or 0) == 0
    want = oracle.conv2d_fused(inp["x"], inp["w"], inp["scale"], inp["shift"], inp["bias"], inp["residual"],
                               stride=(sh.stride,) * 2, pad=(sh.pad,) * 2, relu=True)
    check(to_host(y), want, "bf16", sh.name)
    return y


@pytest.mark.gpu
def test_packed_weights_beyond_the_static_scratch(tvg):
    import torch
    sh = ti.ConvShape("deep", 1, 2052, 7, 7, 1024, 3, 3, 1, 1)
    d = tvg.ConvDesc(1, 2052, 7, 7, 1024, 3, 3, 1, 1, 1, 1, BF16, tvg.TVG_RELU)
    need, least = tvg.tvg_conv2d_workspace_size(d), generic_workspace(d)
    assert 0 < least < tvg.tvg_static_scratch_bytes() < need
    static = _run(tvg, sh, None, static=True)
    assert torch.equal(static, _run(tvg, sh, least))            # both on the generic kernel
    assert torch.equal(static, _run(tvg, sh, need - 1))
    assert torch.equal(_run(tvg, sh, need), _run(tvg, sh, need + 512))


@pytest.mark.gpu
def test_a_short_and_a_misaligned_workspace(tvg):
    import torch
    sh = ti.ConvShape("wide", 8, 45, 65, 63, 60, 3, 3, 1, 1)    # the generic kernel needs none
    d = tvg.ConvDesc(8, 45, 65, 63, 60, 3, 3, 1, 1, 1, 1, BF16, tvg.TVG_RELU)
    need = tvg.tvg_conv2d_workspace_size(d)
    assert need > 0 and generic_workspace(d) == 0
    y = _run(tvg, sh, None)
    assert torch.equal(y, _run(tvg, sh, need - 1)) and torch.equal(y, _run(tvg, sh, need, offset=64))
    _run(tvg, sh, need)


@pytest.mark.gpu
def test_a_block_with_room_for_the_partial_sums_only(tvg):
    import torch
    n, c, hw, k = 1, 1021, 5, 300
    desc, t, least = block(n, c, hw, k)
    dwi = ti.make_inputs(ti.ConvShape("dw", n, c, hw, hw, c, 3, 3, 1, 1, depthwise=True), 6600, "bf16")
    pwi = ti.make_inputs(ti.ConvShape("pw", n, c, hw, hw, k, 1, 1, 1, 0), 6601, "bf16", residual=True, bias=True)
    a, b = dev_inputs(dwi, "bf16"), dev_inputs(pwi, "bf16")
    want = oracle.dwpw_fused(dwi["x"], dwi["w"], dwi["scale"], dwi["shift"], pwi["w"], pwi["scale"], pwi["shift"],
                             pwi["bias"], pwi["residual"], stride=1, relu_dw=True, relu_pw=False)
    for nbytes in (t + least, tvg.tvg_dwpw_workspace_size(desc, k)):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        y = torch.full((n, k, hw, hw), float("nan"), dtype=torch.bfloat16, device="cuda")
        assert tvg.tvg_dwpw_fused(desc, k, 0, a["x"], a["w"], a["scale"], a["shift"], b["w"], b["scale"], b["shift"],
                                  b["bias"], b["residual"], y, ws, nbytes) == 0
        check(to_host(y), want, "bf16", nbytes, tight=BLOCK_TIGHT)
