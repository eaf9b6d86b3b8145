"""One set of trials serves a size and occupancy class, whatever the precision and
the caller: a call whose class has been timed already queues its work and
returns, while trials wait for the stream (here for work queued before them)."""
import numpy as np
import pytest

from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu


def _system(side, seed):
    rng = np.random.default_rng(seed)
    n = 2 * side ** 3
    x, y, z = (rng.integers(0, side << 12, n).astype(np.float32) * 2.0 ** -12 for _ in range(3))
    return synth.System("class", x, y, z, synth._weights(rng, n), (0.0, 0.0, 0.0), (side,) * 3, 1.0, 1.0)


def _returns_at_once(ds, call):
    """Whether `call` comes back while work queued before it still runs."""
    import torch
    busy = torch.cuda.Event()
    for _ in range(400):  # about 0.1 s
        ds.interact(sweep="nolds")
    busy.record()
    call()
    pending = not busy.query()
    ds.sync()
    return pending


def _warm(call_of):
    """The kernels of the call loaded, on a system of another class."""
    from paper_2406_16091_amd import device
    ds = device.DeviceSystem(_system(12, 1))
    ds.bin()
    z = np.zeros(ds.sys.n, np.float32)
    ds.set_velocity(z, z, z)
    call_of(ds)()
    ds.sync()
    ds.close()


def test_a_tuned_sweep_serves_the_time_steps():
    from paper_2406_16091_amd import device, pi

    def step(ds):
        return lambda: ds.step(0.25, 0.0, 2.0 ** -12)

    _warm(step)
    ds = device.DeviceSystem(_system(50, 2))
    ds.bin()
    z = np.zeros(ds.sys.n, np.float32)
    ds.set_velocity(z, z, z)
    pi.pi_tuner_choice(ds.ctx.handle, ds.cells, pi.PI_PREC_COMPENSATED)
    ds.sync()
    assert _returns_at_once(ds, step(ds))
    ds.close()


def test_a_tuned_sweep_serves_the_other_name_of_its_arithmetic():
    from paper_2406_16091_amd import device

    def sweep(ds):
        return lambda: ds.interact(precision="fp64acc")

    _warm(sweep)
    ds = device.DeviceSystem(_system(53, 3))
    ds.bin()
    ds.interact()
    ds.sync()
    assert _returns_at_once(ds, sweep(ds))
    ds.close()
