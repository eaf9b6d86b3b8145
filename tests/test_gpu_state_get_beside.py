"""Read-backs that may run beside one another keep to their own outputs: on the
per-thread stream, whose one handle is another stream in every thread, and under
capture, whose graph may be launched on any stream.  (Only a read-back on the
object's own stream may use the object's scratch.)"""
import ctypes

import numpy as np
import pytest

from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu

N = 1 << 18
NAMES = ("x", "y", "z", "vx", "vy", "vz", "rho", "gx", "gy", "gz")
PER_THREAD = 2  # hipStreamPerThread


def _stepped(stream):
    from paper_2406_16091_amd import device
    s = synth.box_system(N, 40, 11, 16)
    ds = device.DeviceSystem(s)
    ds.bin(stream)
    rng = np.random.default_rng(3)
    ds.set_velocity(*(rng.normal(0, 0.05, N).astype(np.float32) for _ in range(3)), stream)
    ds.step(0.25, 0.02, 2.0 ** -16, stream=stream)
    ds.sync(stream)
    return ds


def _outputs():
    import torch
    return {k: torch.full((N,), 7.0, device="cuda") for k in NAMES}


def test_per_thread_stream():
    import torch
    from paper_2406_16091_amd import pi

    ds = _stepped(PER_THREAD)
    ctx, out = ds.ctx.handle, _outputs()
    torch.cuda.synchronize()
    pi.pi_timing_reset(ctx)
    pi.pi_timing_enable(ctx, True)
    pi.pi_state_get(ctx, ds.cells, *out.values(), PER_THREAD)
    ds.sync(PER_THREAD)
    pi.pi_timing_enable(ctx, False)
    assert set(pi.pi_timing_read(ctx)) == {"k_scatter_state", "k_scatter_forces"}
    ref = ds.state(forces=True)
    for k in NAMES:
        assert np.array_equal(out[k].cpu().numpy(), ref[k]), k
    ds.close()


def test_under_capture():
    import torch
    from paper_2406_16091_amd import device, pi

    s = torch.cuda.Stream()
    ds = _stepped(s)
    ctx, out = ds.ctx.handle, _outputs()
    ref = _outputs()
    torch.cuda.synchronize()
    pi.pi_state_get(ctx, ds.cells, *ref.values(), s)
    torch.cuda.synchronize()
    ds.binned()  # (loads the HIP runtime's handle)
    hip = device._hip
    graph, exe, count = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_size_t()
    st = ctypes.c_void_p(s.cuda_stream)
    assert hip.hipStreamBeginCapture(st, 2) == 0  # relaxed
    pi.pi_state_get(ctx, ds.cells, *out.values(), s)
    assert hip.hipStreamEndCapture(st, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    assert count.value == 2, "one kernel for the state, one for the forces"
    assert hip.hipGraphInstantiate(ctypes.byref(exe), graph, None, None, ctypes.c_size_t(0)) == 0
    other = torch.cuda.Stream()
    for rep in range(4):  # the graph beside an eager read-back on the object's stream
        eager = _outputs()
        for v in out.values():
            v.fill_(-1.0)
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(exe, ctypes.c_void_p(other.cuda_stream)) == 0
        pi.pi_state_get(ctx, ds.cells, *eager.values(), s)
        torch.cuda.synchronize()
        for k in NAMES:
            assert torch.equal(out[k], ref[k]) and torch.equal(eager[k], ref[k]), (rep, k)
    hip.hipGraphExecDestroy(exe)
    hip.hipGraphDestroy(graph)
    ds.close()
