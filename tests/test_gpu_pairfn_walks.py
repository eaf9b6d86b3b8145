"""The no-LDS walk of the pair kernels goes cell by cell only where a launch is too
small to fill the GPU (a large one issues up to 1.4 times as much that way), and
either walk gives the X-pencil's outputs bit for bit."""
import numpy as np
import pytest

from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,side,per_cell,cells", [
    ("lj", 24, 3, True), ("lj", 24, 2, False), ("lj", 26, 11, True), ("lj", 48, 4, False),
    ("lowflop", 20, 20, True), ("lowflop", 40, 8, False),
    ("highflop", 16, 14, True), ("highflop", 16, 13, False), ("highflop", 32, 10, False), ("highflop", 17, 64, True),
])
def test_walk_by_launch_size(kernel, side, per_cell, cells):
    from paper_2406_16091_amd import device, pi

    rng = np.random.default_rng(side)
    n = side ** 3 * per_cell
    x, y, z = (rng.integers(0, side << 12, n).astype(np.float32) * 2.0 ** -12 for _ in range(3))
    s = synth.System("walk", x, y, z, synth._weights(rng, n), (0.0, 0.0, 0.0), (side,) * 3, 1.0, 1.0)
    ds = device.DeviceSystem(s)
    ds.bin()
    ctx = ds.ctx.handle
    out = []
    for sweep in ("pencil", "nolds"):
        pi.pi_timing_reset(ctx)
        pi.pi_timing_enable(ctx, True)
        ds.interact_pairfn(kernel, "compensated", sweep, invariants=False)
        ds.sync()
        pi.pi_timing_enable(ctx, False)
        out.append(ds.results())
    names = set(pi.pi_timing_read(ctx))
    assert names == {"k_pairfn_nolds_cells" if cells else "k_pairfn_nolds"}
    for k in ("rho", "count"):
        assert np.array_equal(out[0][k], out[1][k])
    ds.close()
