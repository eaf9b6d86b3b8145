"""The pair kernels' walks that AUTO and the occupancy pick between -- rows or
cells from global memory, rows staged in LDS -- against each other: the staged
rows only run under AUTO, from 20 per cell and 2^19 particles in static mode.
On lattice inputs every organisation sums the same terms in the same order, so
the outputs equal the X-pencil's bit for bit."""
import numpy as np
import pytest

from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu


def _box(n, dims, clustered, seed=5):
    rng = np.random.default_rng(seed)
    p = [rng.random(n) * d for d in dims]
    if clustered:  # half of the particles in an eighth of each extent: cells of hundreds beside empty ones
        p = [np.where(np.arange(n) % 2 == 0, v / 8.0, v) for v in p]
        empty = p[0] > 0.75 * dims[0]
        p[0] = np.where(empty, p[0] - 0.75 * dims[0], p[0])
    x, y, z = ((np.floor(v * 4096.0) / 4096.0).astype(np.float32) for v in p)
    return synth.System("box", x, y, z, synth._weights(rng, n), (0.0, 0.0, 0.0), dims, 1.0, 1.0)


@pytest.mark.parametrize("kernel", ["lj", "lowflop"])
@pytest.mark.parametrize("precision", ["plain", "compensated"])
@pytest.mark.parametrize("n,dims,clustered", [((1 << 19) + 13, (29, 31, 17), False), (1 << 19, (1, 64, 130), False),
                                              ((1 << 19) + 200, (37, 23, 29), True), (1 << 19, (5003, 3, 1), False)])
def test_staged_rows_equal_the_pencils(kernel, precision, n, dims, clustered):
    from paper_2406_16091_amd import device, pi

    s = _box(n, dims, clustered)
    ctx = device.Context(0)  # a context of its own, in static mode
    pi.pi_tuner_mode(ctx.handle, pi.PI_TUNE_STATIC)
    ds = device.DeviceSystem(s, ctx=ctx)
    ds.bin()
    out = []
    for sweep in ("pencil", "nolds", "auto"):
        ds.interact_pairfn(kernel, precision, sweep, "original", invariants=True)
        ds.sync()
        r, inv = ds.results(), ds.invariants()
        out.append((r["rho"], r["count"], inv["pairs"]))
    for v, c, pairs in out[1:]:
        assert np.array_equal(v, out[0][0]) and np.array_equal(c, out[0][1]) and pairs == out[0][2]
    assert out[0][2] == int(out[0][1].astype(np.int64).sum())
    ds.close()


@pytest.mark.parametrize("n,dims", [(7000, (11, 13, 17)), (20000, (11, 13, 17)), (60000, (19, 13, 17))])
@pytest.mark.parametrize("kernel", ["lj", "highflop"])
def test_cell_and_row_walks_equal_the_pencils(kernel, n, dims):
    from paper_2406_16091_amd import device

    ds = device.DeviceSystem(_box(n, dims, False))
    ds.bin()
    out = []
    for sweep in ("pencil", "nolds"):
        ds.interact_pairfn(kernel, "compensated", sweep, "original", e0=0.75)
        ds.sync()
        out.append(ds.results())
    assert np.array_equal(out[0]["rho"], out[1]["rho"]) and np.array_equal(out[0]["count"], out[1]["count"])
    ds.close()
