"""AUTO on few particles in dense cores: tiles whose densest cell is far above the
mean leave all targets to the dense pass, so that the sweep waits for one chain of a
core's wavefront and not for two; uniform particles stay in the tiles; outputs are the
no-LDS walk's either way."""
import numpy as np
import pytest

from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu

OUT = ("rho", "gx", "gy", "gz", "count")


def _system(n, per, blobs, seed=1):
    """Nine in ten particles in `blobs` blobs, on a 2^-10 lattice."""
    rng = np.random.default_rng(seed)
    side = max(3, round((n / per) ** (1 / 3)))
    p = rng.random((n, 3)) * side
    if blobs:
        q = (rng.random((blobs, 3)) * side)[rng.integers(0, blobs, n)] + 0.05 * side * rng.standard_normal((n, 3))
        p = np.where(rng.random((n, 1)) < 0.1, p, q)
    p = np.floor(np.clip(p, 0, side - 2.0 ** -10) * 1024) / 1024
    x, y, z = p.T.astype(np.float32)
    return synth.System("blobs", x, y, z, synth._weights(rng, n), (0.0, 0.0, 0.0), (side,) * 3, 1.0, 1.0)


@pytest.mark.parametrize("n,per,blobs", [(2 ** 13, 6, 8), (2 ** 13 + 5, 12, 8), (2 ** 16, 8, 8), (2 ** 16 + 1, 8, 8),
                                         (2 ** 13, 5, 8), (2 ** 13, 6, 0), (4, 0.1, 0)])
def test_few_particles_in_dense_cores(n, per, blobs):
    from paper_2406_16091_amd import device, pi

    ctx = device.Context.get(0).handle
    s = _system(n, per, blobs)
    ds = device.DeviceSystem(s)
    ds.bin()
    pi.pi_tuner_mode(ctx, pi.PI_TUNE_STATIC)
    try:
        got = []
        for sweep in ("nolds", "auto", "auto"):
            pi.pi_timing_reset(ctx)
            pi.pi_timing_enable(ctx, True)
            ds.interact(sweep=sweep)
            ds.sync()
            times = pi.pi_timing_read(ctx)
            pi.pi_timing_enable(ctx, False)
            got.append((ds.results(), ds.invariants()["pairs"]))
    finally:
        pi.pi_timing_enable(ctx, False)
        pi.pi_tuner_mode(ctx, pi.PI_TUNE_TIMED)
    ds.close()
    for res, pairs in got[1:]:
        assert pairs == got[0][1]
        for k in OUT:
            assert np.array_equal(res[k], got[0][0][k]), k
    tile = [ms for k, (_, ms) in times.items() if k.startswith("k_sweep_tile")]
    dense = [ms for k, (_, ms) in times.items() if k == "k_sweep_dense"]
    assert len(tile) == len(dense) == 1
    if blobs and n >= 6 * s.dims[0] ** 3 and n <= 2 ** 16:
        assert tile[0] < 0.25 * dense[0], (tile, dense)
    if not blobs:
        assert dense[0] < 0.015, (tile, dense)
