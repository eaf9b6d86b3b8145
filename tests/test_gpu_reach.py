"""Neighbour cells are left out only where no source of theirs can be inside the
cutoff.  The cell of a particle is a float32 decision, so far along a grid whose
cell width is no power of two a particle may lie a little below its cell's low
face; every organisation counts it for targets that its cell's face alone would
put out of reach."""
import numpy as np
import pytest

import oracle
from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu

ORGANISATIONS = [("nolds", (0, 0, 0)), ("stream", (0, 0, 0)), ("subbox", (4, 4, 4)), ("subbox", (6, 6, 6)),
                 ("pencil", (30, 1, 1)), ("pencil", (254, 1, 1)), ("pencilreg", (4, 4, 2)), ("cell", (4, 1, 1)),
                 ("cell", (2, 16, 1))]


def long_system(axis, cells=(1 << 17) + 40, n=3000, seed=5):
    """Particles on one line along `axis`, in the last 60 of a long row of cells; every
    distance is a multiple of 2^-6 and none within 10^-3 of the cutoff."""
    rng = np.random.default_rng(seed)
    w = float(np.float32(1.0012869834899902))
    at = np.floor(rng.uniform((cells - 60) * w, (cells - 0.5) * w, n) * 64) / 64
    c = [np.full(n, 0.5, np.float32) for _ in range(3)]
    c[axis] = at.astype(np.float32)
    dims = [1, 1, 1]
    dims[axis] = cells
    return synth.System("long", *c, synth._weights(rng, n), (0.0, 0.0, 0.0), tuple(dims), w, w)


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_long_rows_count_every_pair(axis):
    from paper_2406_16091_amd import device

    s = long_system(axis)
    b = oracle.bin_particles(s.x, s.y, s.z, s.w, s.origin, s.dims, s.cell_w, s.rc)
    want = oracle.sweep(s.x, s.y, s.z, s.w, s.dims, s.rc, b).count
    ds = device.DeviceSystem(s)
    ds.bin()
    for sweep, tile in ORGANISATIONS:
        ds.interact(sweep=sweep, tile=tile, order="original")
        ds.sync()
        wrong = ds.results()["count"].astype(np.int64) - want
        assert not wrong.any(), (sweep, tile, int((wrong != 0).sum()), int(wrong.sum()))
    ds.close()
