"""The native call path from Python (csrc/native_calls.cpp) away from its ordinary case, on the GPU."""
import pytest

pytestmark = pytest.mark.gpu


def test_an_output_that_does_not_fit_raises_out_of_memory(tvg):
    """torch's own exception type, as from torch.empty, so that programs that catch it (to split a batch)
    go on working.  y is 1.2 GB under a limit of 1/256 of the card's memory."""
    import torch
    x = torch.zeros((4, 1, 1024, 1024), device="cuda")
    w = torch.zeros((75, 1, 1, 1), device="cuda")
    s = torch.ones(75, device="cuda")
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(1.0 / 256)
    try:
        with pytest.raises(torch.cuda.OutOfMemoryError):
            tvg.conv2d_fused(x, w, s, s)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
