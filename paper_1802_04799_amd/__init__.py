"""Python binding of libtvg: fused conv2d / depthwise conv2d for one MI355X (gfx950).

Argument marshalling only; every operator runs in the HIP kernels of
``libtvg.so`` (C ABI declared in ``include/tvg.h``).  PyTorch supplies device
memory and streams.  There is no CPU fallback: if the library is missing,
``load()`` raises.
"""
from . import binding as _binding
from .binding import (  # noqa: F401
    TVG_BF16, TVG_F32, TVG_RELU, TVG_STREAM_OUT, ConvDesc, TvgError, lib_path, load,
    maxpool2d_3x3s2, status_string, tvg_conv2d_workspace_size,
    tvg_dwconv2d_workspace_size, tvg_version,
    KERNEL_NAMES, tvg_conv2d_get_plan, tvg_conv2d_set_tile, ConvKnobs, tvg_conv2d_set_knobs, tvg_conv2d_get_knobs,
    tvg_static_scratch_bytes, tvg_conv2d_prepack_size, tvg_conv2d_prepack,
    tvg_probe_copy, tvg_probe_mfma, TVG_CENTRE_TAP_ONLY,
    TensorLife, tvg_plan_arena, tvg_dwpw_one_kernel, tvg_dwpw_workspace_size,
)


def __getattr__(name):
    # the operator calls (binding.NATIVE_NAMES): resolved on first use, see binding.native()
    if name in _binding.NATIVE_NAMES:
        fn = getattr(_binding, name)
        if name in vars(_binding):           # (resolved for good)
            globals()[name] = fn
        return fn
    raise AttributeError(f"module {__name__!r} has no attribute {name!r}")


def __dir__():
    return sorted(set(globals()) | set(_binding.NATIVE_NAMES))


__all__ = [_n for _n in globals() if not _n.startswith("_")] + list(_binding.NATIVE_NAMES)
