"""Read-backs on another stream than the step's are ordered as work on that
stream is: a blocking stream and the null stream wait for each other's work by
themselves, so the results are those of the step that the other of the two
still runs, after mhd_set_stream and after a graph replayed there.
"""
import ctypes

import pytest

from paper_2510_24175_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture
def blocking_stream():
    """A stream from hipStreamCreate of the runtime that the library is linked
    to (torch's own streams do not block)."""
    import torch

    from paper_2510_24175_amd import mhd

    lib = mhd.load_library()
    handle = ctypes.c_void_p()
    torch.cuda.synchronize()
    assert lib.hipStreamCreate(ctypes.byref(handle)) == 0
    yield torch.cuda.ExternalStream(handle.value)
    torch.cuda.synchronize()
    lib.hipStreamDestroy(handle)


def steps(ctx, V):
    """Two states and the results of a step from each."""
    import torch

    A = ctx.prim_to_cons(torch.from_numpy(V).cuda())
    torch.cuda.synchronize()
    B, C = torch.empty_like(A), torch.empty_like(A)
    dt, ch = ctx.cfl_dt(A)
    ctx.step(A, B, dt, ch)
    first = ctx.step_info()
    ctx.step(B, C, dt, ch)
    second = ctx.step_info()
    assert first != second
    return A, B, C, dt, ch, first, second


@pytest.mark.parametrize("first", ["null", "blocking"])
def test_results_across_streams(first, blocking_stream):
    import torch

    from paper_2510_24175_amd.mhd import Context

    setup, V = W.turbulence(256)
    ctx = Context(setup, "f32", stream=torch.cuda.default_stream())
    streams = [torch.cuda.default_stream(), blocking_stream]
    if first == "blocking":
        streams.reverse()
    A, B, C, dt, ch, old, want = steps(ctx, V)
    ctx.step(A, C, dt, ch)
    assert ctx.step_info() == old
    ctx.set_stream(streams[0])
    for _ in range(4):  # the results are those of the last step
        ctx.step(A, C, dt, ch)
    ctx.step(B, C, dt, ch)
    ctx.set_stream(streams[1])
    assert ctx.step_info() == want
    torch.cuda.synchronize()
    assert ctx.step_info() == want
    ctx.close()


def test_results_of_a_graph_replayed_elsewhere(blocking_stream):
    import torch

    from paper_2510_24175_amd.mhd import Context

    setup, V = W.turbulence(256)
    ctx = Context(setup, "f32", stream=blocking_stream)
    A, B, C, dt, ch, old, want = steps(ctx, V)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=blocking_stream):
        for _ in range(4):
            ctx.step(A, C, dt, ch)
        ctx.step(B, C, dt, ch)
    for _ in range(3):
        ctx.step(A, C, dt, ch)
        assert ctx.step_info() == old
        graph.replay()  # on the null stream
        assert ctx.step_info() == want
    torch.cuda.synchronize()
    ctx.close()
