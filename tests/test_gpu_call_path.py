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


def _calls(tvg, torch):
    """name -> call(out, stream) of every convenience call, natively and (relu=1: not a bool) through the
    Python implementation; the dense shapes pack their weights into a workspace."""
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    r = lambda *s: torch.rand(s, generator=g, device="cuda") * 2 - 1
    b = lambda *s: r(*s).bfloat16()
    x, w, s = b(8, 45, 65, 63), b(60, 45, 3, 3), r(60)
    x2, w2, s2 = b(2, 300, 13, 13), b(31, 300, 5, 5), r(31)
    wd, sd, wp, sp = b(45, 1, 3, 3), r(45), b(60, 45, 1, 1), r(60)
    calls = {}
    for kind, yes in (("native", True), ("python", 1)):
        calls[f"conv2d {kind}"] = lambda out, st, yes=yes: tvg.conv2d_fused(x, w, s, s, pad=1, relu=yes, out=out, stream=st)
        calls[f"conv2d split {kind}"] = lambda out, st, yes=yes: tvg.conv2d_fused(x2, w2, s2, s2, pad=2, relu=yes, out=out, stream=st)
        calls[f"dwconv2d {kind}"] = lambda out, st, yes=yes: tvg.dwconv2d_fused(x, wd, sd, sd, relu=yes, out=out, stream=st)
        calls[f"dwpw {kind}"] = lambda out, st, yes=yes: tvg.dwpw_fused(x, wd, sd, sd, wp, sp, sp, relu_pw=yes, out=out, stream=st)
    calls["maxpool"] = lambda out, st: tvg.maxpool2d_3x3s2(x, out=out, stream=st)
    return calls


@pytest.mark.parametrize("as_handle", [False, True])
def test_a_launch_on_another_stream_takes_its_memory_from_that_streams_pool(tvg, as_handle):
    """torch's allocator hands a freed block out again in the order of the stream it was allocated on: what a
    call allocates for a launch on `stream` must not come back on the current stream while the launch runs."""
    import torch
    for name, call in _calls(tvg, torch).items():
        want = call(None, None)
        assert torch.cuda.current_stream().cuda_stream == 0
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        y = call(None, side.cuda_stream if as_handle else side)
        assert torch.cuda.current_stream().cuda_stream == 0, name
        home = [g for g in torch.cuda.memory_snapshot()
                if g["address"] <= y.data_ptr() < g["address"] + g["total_size"]]
        assert len(home) == 1 and home[0]["stream"] == side.cuda_stream, name
        side.synchronize()
        assert torch.equal(y, want), name
        # the workspace alone (out given): nothing that the current stream's pool could hand out
        torch.cuda.empty_cache()
        before = {g["address"] for g in torch.cuda.memory_snapshot() if g["stream"] == 0}
        torch.cuda.reset_peak_memory_stats()
        call(y, side.cuda_stream if as_handle else side)
        after = {g["address"] for g in torch.cuda.memory_snapshot() if g["stream"] == 0}
        assert after == before, name
        if name.startswith(("conv2d", "dwpw")):
            assert torch.cuda.max_memory_allocated() > torch.cuda.memory_allocated(), name      # (there was one)
        side.synchronize()
        assert torch.equal(y, want), name


def test_calls_on_two_streams_do_not_share_a_workspace(tvg):
    """Two dense calls that pack their weights, on two side streams at once, while the current stream
    allocates and fills memory of the same sizes: the results of the same calls on the current stream."""
    import torch
    calls = _calls(tvg, torch)
    one, two = calls["conv2d native"], calls["conv2d split native"]
    want1, want2 = one(None, None), two(None, None)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    got = []
    for _ in range(20):
        got.append((one(None, a), two(None, b)))
        for nbytes in (65536, 691936, want1.nbytes, want2.nbytes):
            torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    for y1, y2 in got:
        assert torch.equal(y1, want1) and torch.equal(y2, want2)


def test_a_stream_of_the_callers_choice_inside_a_captured_graph(tvg):
    """A side stream that has joined a capture: the call's memory comes from the graph's pool, and every
    replay gives the eager result."""
    import torch
    call = _calls(tvg, torch)["conv2d split native"]
    want = call(None, None)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        side.wait_stream(torch.cuda.current_stream())
        y = call(None, side)
        torch.cuda.current_stream().wait_stream(side)
    for _ in range(4):
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want) and torch.equal(call(None, None), want)


def test_unusual_arguments_get_the_answers_of_the_python_implementation(tvg):
    """A tensor without storage (inside vmap and vjp), a nested stride, a tensor subclass."""
    import torch
    x, w, s = torch.rand(2, 1, 8, 5, 5, device="cuda"), torch.rand(8, 8, 3, 3, device="cuda"), torch.ones(8, device="cuda")
    want = tvg.conv2d_fused(x[0], w, s, s, pad=1)
    o = torch.empty(1, 8, 5, 8, device="cuda")
    for f in (lambda a: tvg.conv2d_fused(a, w, s, s, pad=1, out=o), lambda a: tvg.conv2d_fused(x[0], w, a[0, 0, 0], s, pad=1)):
        for transform in (lambda: torch.vmap(f)(x[..., :1].expand(2, 1, 8, 5, 8).contiguous()),
                          lambda: torch.func.vjp(f, x[0][..., :1].expand(1, 8, 5, 8).contiguous())):
            with pytest.raises(RuntimeError, match="Cannot access data pointer"):
                transform()
    for stride in (((1, 2), 1), (1, (1, 1)), [1], (1, 1, 1), "1", 1.0):
        with pytest.raises((TypeError, ValueError)):
            tvg.conv2d_fused(x[0], w, s, s, pad=1, stride=stride)
    for stride in (1, (1, 1), [1, 1]):
        assert torch.equal(tvg.conv2d_fused(x[0], w, s, s, pad=1, stride=stride), want)

    class Named(torch.Tensor):
        pass

    assert torch.equal(tvg.conv2d_fused(x[0].as_subclass(Named), torch.nn.Parameter(w), s, s, pad=1), want)


def test_outputs_and_workspaces_of_the_callers_own(tvg):
    """Natively: an output on the host, short or strided is refused, a larger one takes the result at its
    start; a strided workspace is not written."""
    import torch
    x, w, s = torch.rand(1, 83, 9, 9, device="cuda").bfloat16(), torch.rand(40, 83, 3, 3, device="cuda").bfloat16(), torch.ones(40, device="cuda")
    want = tvg.conv2d_fused(x, w, s, s, pad=1)
    b = lambda *shape: torch.full(shape, 7.0, dtype=torch.bfloat16, device="cuda")
    for out in (torch.empty(1, 40, 9, 9, dtype=torch.bfloat16), b(1, 40, 9, 8), b(1, 40, 9, 18)[..., ::2], b(1, 40, 9, 1).expand(1, 40, 9, 9)):
        with pytest.raises(ValueError):
            tvg.conv2d_fused(x, w, s, s, pad=1, out=out)
    out = b(2, 40, 9, 9)
    assert tvg.conv2d_fused(x, w, s, s, pad=1, out=out) is out
    assert torch.equal(out[:1], want) and bool((out[1] == 7.0).all())
    ws = torch.full((2, 1 << 20), 9, dtype=torch.uint8, device="cuda").t()
    assert torch.equal(tvg.conv2d_fused(x, w, s, s, pad=1, workspace=ws), want) and bool((ws == 9).all())
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    assert torch.equal(tvg.conv2d_fused(x, w, s, s, pad=1, workspace=ws), want)
    with pytest.raises(ValueError):
        tvg.conv2d_fused(x, w, s, s, pad=1, workspace=ws.cpu())
