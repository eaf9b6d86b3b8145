"""Cell counts around which the radix passes take digits of nine bits: every
binned array bit for bit the oracle's, of one system and of a batch."""
import numpy as np
import pytest

import oracle
from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu


def _check(g, b, off=0, cb=0):
    n, nc = len(b.perm), len(b.counts)
    assert np.array_equal(g["counts"][cb:cb + nc], b.counts)
    assert np.array_equal(g["offsets"][cb:cb + nc + 1] - off, b.offsets)
    assert np.array_equal(g["perm"][off:off + n] - off, b.perm)
    assert np.array_equal(g["cell"][off:off + n], b.cell[b.perm])
    for k in ("xs", "ys", "zs", "ws"):
        assert np.array_equal(g[k][off:off + n].view(np.uint32), getattr(b, k).view(np.uint32)), k


@pytest.mark.parametrize("n,dims", [
    (262145, (16, 16, 1)),      # 8 bits: one pass of 8
    (262145, (257, 1, 1)),      # 9 bits: one of 9
    (270000, (8, 8, 8)),
    (270000, (64, 32, 32)),     # 16 bits: two of 8
    (270000, (1, 65537, 1)),    # 17 bits: two of 9
    (1000000, (64, 64, 64)),
    (270000, (65, 64, 64)),     # 19 bits: three of 8
    (5000, (512, 512, 65)),     # 25 bits: three of 9
])
def test_one_system(n, dims):
    from paper_2406_16091_amd import device

    rng = np.random.default_rng(sum(dims))
    x, y, z = ((rng.integers(0, d * 64, n) / 64).astype(np.float32) for d in dims)
    s = synth.System("digits", x, y, z, rng.random(n, dtype=np.float32), (0.0, 0.0, 0.0), dims, 1.0, 1.0)
    ds = device.DeviceSystem(s)
    ds.bin()
    g = ds.binned()
    b = oracle.bin_particles(x, y, z, s.w, s.origin, dims, 1.0, 1.0)
    _check(g, b)
    assert g["max_per_cell"] == b.max_per_cell


@pytest.mark.parametrize("sides", [(5, 6), (40, 30, 1), (64,), (64, 2)])
def test_batch(sides):
    from paper_2406_16091_amd import device

    systems = [synth.box_system(2000 + 37 * k, g, seed=50 + k, lattice_log2=12) for k, g in enumerate(sides)]
    db = device.DeviceBatch(systems)
    db.run()
    db.sync()
    g = db.binned()
    for i, s in enumerate(systems):
        _check(g, oracle.bin_particles(s.x, s.y, s.z, s.w, s.origin, s.dims, s.cell_w, s.rc), db.offsets[i],
               g["cell_base"][i])
