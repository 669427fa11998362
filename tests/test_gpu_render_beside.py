"""GPU tests of render calls beside what the rest of a program does on the GPU:
a capture that is under way on another stream, and an error that an earlier
call of the program left behind."""
import ctypes
import threading

import pytest

from paper_1209_6038_amd import workloads as W
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu


def _job():
    import torch
    from paper_1209_6038_amd import rt
    cl, cams = [rt.Cloak(W.cloak(1, height=W.HEIGHT))], W.render_views(32, (30.0,))
    ref = rt.render_multi(cl, W.render_opts(), W.room(), cams, 3)
    torch.cuda.synchronize()
    return cl, cams, ref, torch.zeros_like(ref)


@pytest.mark.parametrize("flag", [0, 1])  # the captured stream: ordered with the null stream, or not
@pytest.mark.parametrize("mode", [0, 1, 2])  # global, thread-local, relaxed
@pytest.mark.parametrize("thread", [False, True])
def test_render_on_the_null_stream_beside_a_capture(flag, mode, thread):
    """Another stream's capture neither refuses a render on the null stream nor
    is ended by it."""
    import torch
    from paper_1209_6038_amd import rt
    say(f"case render beside capture flag={flag} mode={mode} thread={thread}")
    hip = ctypes.CDLL("libamdhip64.so")
    cl, cams, ref, out = _job()
    failed = []

    def render():
        try:
            rt.render_multi(cl, W.render_opts(), W.room(), cams, 3, out=out)
        except rt.RtError as e:
            failed.append(str(e))

    stream, graph = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(stream), flag) == 0
    assert hip.hipStreamBeginCapture(stream, mode) == 0
    if thread:
        t = threading.Thread(target=render)
        t.start()
        t.join()
    else:
        render()
    end = hip.hipStreamEndCapture(stream, ctypes.byref(graph))
    hip.hipGetLastError()
    if graph.value:
        hip.hipGraphDestroy(graph)
    torch.cuda.synchronize()
    hip.hipStreamDestroy(stream)
    assert not failed and end == 0
    assert torch.equal(out, ref)


def test_earlier_error_is_not_the_uploads():
    """An error that a call of the program's own left behind neither refuses a
    plan or a launch-shape search nor keeps a render from being made (which
    reports it, as every call that checks its launches does)."""
    import torch
    from paper_1209_6038_amd import rt
    say("case render after an earlier error")
    hip = ctypes.CDLL("libamdhip64.so")
    cl, cams, ref, out = _job()

    def leave_error():
        torch.cuda.synchronize()
        p = ctypes.c_void_p()
        assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(1 << 60)) != 0

    try:
        leave_error()
        with pytest.raises(rt.RtError):
            rt.render_multi(cl, W.render_opts(), W.room(), cams, 3, out=out)
        leave_error()
        plan = rt.RenderPlan(cl, W.render_opts(), W.room(), cams, 3)
        leave_error()
        rt.autotune_render(cl, W.render_opts(), W.room(), cams, 3)
    finally:
        hip.hipGetLastError()
    plan.launch()
    torch.cuda.synchronize()
    assert torch.equal(out, ref) and torch.equal(plan.rgb, ref)
    plan.close()
