"""The native call path from Python (csrc/native_calls.cpp) away from its ordinary case, on a machine
without a GPU: device tensors here are torch's fake ones (shapes and devices, address NULL), so that a
call gets as far as the library's NULL check and no further.  Each case that could end the process runs
in a process of its own."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import warnings; warnings.simplefilter("ignore")
import torch
import paper_1802_04799_amd as tvg
from torch._subclasses.fake_tensor import FakeTensorMode
def dev(*shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device="cuda")
def outcome(f):
    try:
        f()
        print("returned")
    except Exception as e:
        print(type(e).__name__, str(e).splitlines()[0])
with FakeTensorMode(allow_non_fake_inputs=True):
    x, w, s, o = dev(2, 1, 8, 5, 5), dev(8, 8, 3, 3), dev(8), dev(1, 8, 5, 5)
    wd, wp, ws = dev(8, 1, 3, 3), dev(8, 8, 1, 1), dev(1 << 16, dtype=torch.uint8)
"""


def outcome(body):
    """What a fresh process prints for `body`, which runs under the fake mode."""
    code = PRELUDE + "".join("    " + line + "\n" for line in body.strip().splitlines())
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
    return r.stdout.strip().splitlines()


@pytest.mark.parametrize("call", [
    "tvg.conv2d_fused(a, w, s, s, pad=1, out=o, stream=0)",
    "tvg.dwconv2d_fused(a, wd, s, s, pad=1, out=o, stream=0)",
    "tvg.dwpw_fused(a, wd, s, s, wp, s, s, out=o, workspace=ws, stream=0)",
])
@pytest.mark.parametrize("transform", ["torch.vmap(f)(x)", "torch.func.vjp(f, x[0])", "torch.func.jvp(f, (x[0],), (x[0],))"])
def test_a_tensor_without_storage_is_a_python_exception(call, transform):
    """Inside vmap, vjp and jvp an operand has no address: torch raises when it is asked for, as it did
    for the Python implementation of these calls, and the process lives on."""
    got = outcome(f"f = lambda a: {call}\noutcome(lambda: {transform})")
    assert len(got) == 1 and got[0].startswith("RuntimeError Cannot access data pointer"), got


def test_star_import_holds_the_operator_calls():
    names = ["conv2d_fused", "dwconv2d_fused", "dwpw_fused", "maxpool2d_3x3s2", "tvg_conv2d_fused", "tvg_dwconv2d_fused",
             "tvg_conv2d_fused_static", "tvg_conv2d_fused_dual", "tvg_conv2d_fused_prepacked", "tvg_dwpw_fused",
             "tvg_maxpool2d_3x3s2", "ConvDesc", "TvgError", "TVG_BF16", "tvg_conv2d_get_plan", "binding"]
    for module in ("paper_1802_04799_amd", "paper_1802_04799_amd.binding"):
        scope = {}
        exec(f"from {module} import *", scope)
        assert [n for n in names if n not in scope and (n != "binding" or "." not in module)] == []


def _plain(code):
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout.split()


def test_raw_calls_with_integer_addresses_need_no_torch():
    """NULL addresses and descriptors that fail: the library's answers, through ctypes."""
    assert _plain("""
import sys; sys.modules["torch"] = None
import paper_1802_04799_amd as tvg
d = tvg.ConvDesc(1, 8, 10, 10, 8, 3, 3, 1, 1, 1, 1, 0, 0)
n = tvg.ConvDesc(0, 8, 10, 10, 8, 3, 3, 1, 1, 1, 1, 0, 0)
print(tvg.tvg_conv2d_fused(d, 4096, None, 4096, 4096, None, None, 4096, None, 0, 0),
      tvg.tvg_conv2d_fused(n, 4096, 4096, 4096, 4096, None, None, y=4096, stream=0),
      tvg.tvg_conv2d_fused_dual(d, 4.0, 8, 0, 0, 0, 0, None, None, 0, 0, 0),
      tvg.tvg_conv2d_fused_prepacked(d, 0, 0, 0, 0, None, None, 0, 0, 0, 0),
      tvg.tvg_dwpw_fused(d, 8.0, 0, *[None] * 10, stream=0),
      tvg.tvg_maxpool2d_3x3s2(1, 1, 0, 4, 0, 4096, 4096, 0))
for wrong in (lambda: tvg.tvg_maxpool2d_3x3s2(1, 1, 4, 4, 0, 0), lambda: tvg.tvg_maxpool2d_3x3s2(1, 1, 4, 4, 0, 0, 0, 0, nope=1),
              lambda: tvg.tvg_maxpool2d_3x3s2(1, 1, 4, 4, 0, 0, 0, 0, n=1)):
    try:
        wrong()
    except TypeError:
        print("TypeError")
""") == ["1", "2", "3", "3", "1", "2"] + ["TypeError"] * 3


def test_names_resolve_and_calls_fail_loudly_without_the_library():
    assert _plain("""
import paper_1802_04799_amd.binding as b
b._LIB_PATH = "/nowhere/libtvg.so"
import paper_1802_04799_amd as tvg
from paper_1802_04799_amd import *
for call in (lambda: conv2d_fused(*[__import__("torch").zeros(1, 1, 1, 1)] * 4), lambda: tvg.tvg_conv2d_fused(*[None] * 8)):
    try:
        call()
    except (ImportError, ValueError) as e:
        print(type(e).__name__)
""") == ["ValueError", "ImportError"]


def test_integers_are_taken_as_before():
    import paper_1802_04799_amd as tvg
    d = tvg.ConvDesc(1, 8, 10, 10, 8, 3, 3, 1, 1, 1, 1, 0, 0)
    assert tvg.tvg_dwpw_fused(d, 8.0, 0.0, *[None] * 10, stream=0) == 1             # int() of what is given
    assert tvg.tvg_conv2d_fused_dual(d, "4", 8.0, 0, 0, 0, 0, None, None, 0, 0, 0) == 3
    assert tvg.tvg_conv2d_fused(d, *[None] * 7, None, 2**64 - 1, 0) == 1            # size_t
    for call in (lambda: tvg.tvg_maxpool2d_3x3s2(1.0, 1, 4, 4, 0, None, None, 0),
                 lambda: tvg.tvg_conv2d_fused(d, *[None] * 7, None, 1.5, 0)):
        with pytest.raises(TypeError):
            call()


def test_a_tensor_subclass_is_asked_for_its_address():
    import torch
    import paper_1802_04799_amd as tvg

    class Guarded(torch.Tensor):
        def data_ptr(self):
            raise LookupError("no address for you")

    t = torch.zeros(1, 8, 5, 5).as_subclass(Guarded)
    d = tvg.ConvDesc(1, 8, 5, 5, 8, 3, 3, 1, 1, 1, 1, 0, 0)
    with pytest.raises(LookupError):
        tvg.tvg_conv2d_fused(d, t, None, None, None, None, None, None, None, 0, 0)


@pytest.mark.parametrize("call,k", [("tvg.conv2d_fused(x[0], w, s, s, pad=1, out=OUT, stream=0)", 8),
                                    ("tvg.dwconv2d_fused(x[0], wd, s, s, pad=1, out=OUT, stream=0)", 8),
                                    ("tvg.dwpw_fused(x[0], wd, s, s, wp, s, s, out=OUT, workspace=ws, stream=0)", 8),
                                    ("tvg.maxpool2d_3x3s2(x[0], out=OUT, stream=0)", 8)])
def test_an_output_the_kernel_must_not_write_is_refused(call, k):
    """On the host, short, strided or overlapping: an exception before any launch; a larger one, or one of
    another type that holds the bytes, is taken (and gets as far as the NULL address)."""
    outs = {"torch.empty(1, 8, 5, 5)": "must be a device tensor", "dev(1, 8, 2, 4)": "too small",
            "dev(1, 8, 5, 10)[..., ::2]": "must be contiguous", "dev(1, 8, 5, 1).expand(1, 8, 5, 5)": "must be contiguous",
            "dev(800, dtype=torch.uint8)": "NULL", "dev(4, 8, 5, 5)": "NULL"}
    got = outcome("\n".join(f"outcome(lambda: {call.replace('OUT', o)})" for o in outs))
    assert len(got) == len(outs)
    for (o, want), line in zip(outs.items(), got):
        assert want in line and line.startswith("TvgError" if want == "NULL" else "ValueError"), (o, line)


def test_a_workspace_on_the_host_is_refused():
    got = outcome("""
b = lambda *s: dev(*s, dtype=torch.bfloat16)
xr, wr, o = b(1, 83, 45, 37), b(139, 83, 3, 3), b(1, 139, 45, 37)
sr = dev(139)
for ws in (torch.empty(1 << 24, dtype=torch.uint8), dev(1 << 24, dtype=torch.uint8)):
    outcome(lambda: tvg.conv2d_fused(xr, wr, sr, sr, pad=1, out=o, workspace=ws, stream=0))
outcome(lambda: tvg.conv2d_fused(x[0], w, s, s, pad=1, out=dev(1, 8, 5, 5), workspace=torch.empty(9), stream=0))
outcome(lambda: tvg.dwpw_fused(x[0], wd, s, s, wp, s, s, out=dev(1, 8, 5, 5), workspace=torch.empty(1 << 16), stream=0))
""")
    assert [line.split()[0] for line in got] == ["ValueError", "TvgError", "TvgError", "ValueError"], got
