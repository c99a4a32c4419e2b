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
