"""pi_state_get around the size from which it goes through 16-byte records, and
on another stream than the object's, where it scatters directly: the same bits,
whichever groups of outputs are asked for."""
import numpy as np
import pytest

from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(1 << 18) - 1, 1 << 18, (1 << 18) + 77])
def test_read_back_paths_agree(n):
    import torch
    from paper_2406_16091_amd import device, pi

    s = synth.box_system(n, 40, 11, 16)
    ds = device.DeviceSystem(s)
    ds.bin()
    rng = np.random.default_rng(3)
    ds.set_velocity(*(rng.normal(0, 0.05, n).astype(np.float32) for _ in range(3)))
    for _ in range(2):
        ds.step(0.25, 0.02, 2.0 ** -16)
    ds.sync()
    other = torch.cuda.Stream()
    names = ("x", "y", "z", "vx", "vy", "vz", "rho", "gx", "gy", "gz")

    def get(groups, stream):
        out = {k: torch.full((n,), 7.0, device="cuda") for k in names}
        keep = [k for i, k in enumerate(names) if min(i // 3, 2) in groups]
        torch.cuda.synchronize()
        pi.pi_state_get(ds.ctx.handle, ds.cells, *(out[k] if k in keep else None for k in names), stream)
        torch.cuda.synchronize()
        return {k: out[k].cpu().numpy() for k in names}, keep

    ref, _ = get((0, 1, 2), other)
    for groups in ((0, 1, 2), (0,), (1,), (2,), (0, 2)):
        got, keep = get(groups, None)
        for k in names:
            assert np.array_equal(got[k], ref[k] if k in keep else np.full(n, 7.0, np.float32)), (groups, k)
    # the records left the binned system as it was: the next step is the same
    got = ds.state(forces=True)
    for k in names:
        assert np.array_equal(got[k], ref[k])
    ds.close()
