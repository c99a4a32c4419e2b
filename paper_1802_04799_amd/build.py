"""Builds libtvg.so (HIP, gfx950 only) and the binding's extension module _native.so next to this
file with hipcc and g++.

Run as ``python -m paper_1802_04799_amd.build``; ``build(force=True)`` recompiles
every source.  The library is built in-tree so that it travels with the
repository snapshot to the GPU machine.
"""
from __future__ import annotations

import importlib.util
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libtvg.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["api.cpp", "conv_igemm.hip", "conv3x3_patch.hip", "conv3x3_dbuf.hip", "conv7x7s2_stem.hip", "conv1x1.hip", "dwconv.hip", "dwpw.hip", "pool.hip", "probe.hip", "conv_f32_small.hip", "conv3x3_winograd.hip", "conv1x1_deep.hip", "conv_bf16_any.hip", "conv_f32_tiled.hip", "conv_rows.hip", "conv_f32_pw.hip", "conv1x1_rows.hip", "conv3x3_strips.hip"]
HEADERS = [os.path.join(CSRC, "tvg_internal.h"), os.path.join(CSRC, "tvg_device.h"),
           os.path.join(ROOT, "include", "tvg.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-x", "hip",
         # packed-fp32 instruction forms are disabled for every device function
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _stale(target: str, deps) -> bool:
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def _compile(src: str, force: bool) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    path = os.path.join(CSRC, src)
    if force or _stale(obj, [path] + HEADERS):
        cmd = [HIPCC] + FLAGS + ["-c", path, "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
        warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if warn.strip():
            sys.stderr.write(warn + "\n")
    return obj


def _torch_dir() -> str:
    """torch's installation folder, found without importing it."""
    spec = importlib.util.find_spec("torch")
    if spec is None:
        raise RuntimeError("the binding's extension module needs torch's headers and libraries")
    return os.path.dirname(spec.origin)


def _build_native(force: bool) -> None:
    """The Python call path: plain C++ against torch's headers, linked to libtvg.so beside it."""
    src = os.path.join(CSRC, "native_calls.cpp")
    if not force and not _stale(NATIVE, [src, LIB, os.path.join(ROOT, "include", "tvg.h")]):
        return
    t = _torch_dir()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-I", os.path.join(ROOT, "include"),
           "-isystem", os.path.join(t, "include"), "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"),
           "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"], src, "-o", NATIVE,
           "-L", HERE, "-ltvg", "-L", os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10",
           "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"building {NATIVE} failed:\n{r.stdout}\n{r.stderr}")
    if r.stderr.strip():
        sys.stderr.write(r.stderr)


def build(force: bool = False, verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=4) as pool:
        objs = list(pool.map(lambda s: _compile(s, force), SOURCES))
    if force or _stale(LIB, objs):
        cmd = [HIPCC, "-shared", "--offload-arch=gfx950", "-o", LIB] + objs + \
              ["-Wl,-rpath,/opt/rocm/lib"]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    _build_native(force)
    if verbose:
        print("built", LIB, NATIVE)
    return LIB


if __name__ == "__main__":
    build(force="--force" in sys.argv, verbose=True)
