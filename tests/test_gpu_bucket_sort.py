"""Binning of few particles (one workgroup, or one radix pass and a workgroup
per bucket of cells) and the sizes at which it hands over to the radix passes:
every array bit for bit the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # n, cells per axis, fraction of each axis that holds the particles
    (1, (1, 1, 1), (1, 1, 1)),
    (4096, (16, 16, 16), (1, 1, 1)),  # the most for one workgroup: particles
    (4097, (16, 16, 16), (1, 1, 1)),
    (4096, (17, 16, 16), (1, 1, 1)),  # and cells
    (4096, (3, 5, 7), (1, 1, 1)),     # dense cells
    (4097, (6, 6, 6), (1, 1, 1)),     # too few cells for buckets
    (8192, (8, 8, 8), (1, 1, 1)),     # buckets of two cells
    (65536, (8, 8, 8), (1, 1, 1)),    # of 128 particles each
    (5000, (10, 11, 13), (1, 1, 1)),
    (65536, (64, 64, 64), (1, 1, 1)),  # the most tiles that sum the digit counts themselves
    (65537, (64, 64, 64), (1, 1, 1)),
    (262144, (64, 64, 64), (1, 1, 1)),  # the most for one pass: particles
    (262145, (64, 64, 64), (1, 1, 1)),
    (5000, (128, 128, 64), (1, 1, 1)),  # and cells
    (5000, (128, 128, 65), (1, 1, 1)),
    (4096, (128, 128, 32), (1, 1 / 8, 1 / 32)),  # one bucket of 2^11 cells, the largest that
    (4097, (128, 128, 32), (1, 1 / 8, 1 / 32)),  # is ranked by comparison, and one more
    (4500, (128, 128, 64), (1, 1 / 4, 1 / 64)),  # 2^12 cells: eight wavefronts' counters
    (65536, (32, 32, 32), (1, 1, 1 / 32)),       # a layer: 64 per cell
    (65536, (64, 64, 32), (1 / 64, 1 / 64, 1 / 32)),  # everything in one cell
    (30000, (64, 64, 32), (1 / 8, 1 / 32, 1 / 32)),   # in eight cells of one bucket
]


@pytest.mark.parametrize("n,dims,part", CASES)
def test_small_binnings_equal_the_oracle(n, dims, part):
    from paper_2406_16091_amd import device

    rng = np.random.default_rng(n + sum(dims))
    x, y, z = ((rng.integers(0, max(int(d * f * 1024), 1), n) / 1024).astype(np.float32) for d, f in zip(dims, part))
    w = rng.random(n, dtype=np.float32)
    s = synth.System("few", x, y, z, w, (0.0, 0.0, 0.0), dims, 1.0, 1.0)
    b = oracle.bin_particles(x, y, z, w, s.origin, dims, 1.0, 1.0)
    ds = device.DeviceSystem(s)
    for _ in range(2):  # buffers of a previous binning
        ds.bin()
    g = ds.binned()
    for k in ("counts", "offsets", "perm"):
        assert np.array_equal(g[k], getattr(b, k)), k
    assert np.array_equal(g["cell"], b.cell[b.perm])
    for k in ("xs", "ys", "zs", "ws"):
        assert np.array_equal(g[k].view(np.uint32), getattr(b, k).view(np.uint32)), k
    assert g["max_per_cell"] == b.max_per_cell


@pytest.mark.parametrize("n", [64, 65])
def test_cells_at_the_comparison_limit(n):
    """A bucket whose fullest cell holds 64 particles, or one more."""
    from paper_2406_16091_amd import device

    rng = np.random.default_rng(n)
    m = 5000
    x, y, z = (rng.integers(0, 32 * 64, m).astype(np.float32) / 64 for _ in range(3))
    pick = rng.permutation(m)[:n]
    x[pick], y[pick], z[pick] = 3.5, 4.25, 5.0
    keep = np.ones(m, bool)
    keep[(np.floor(x) == 3) & (np.floor(y) == 4) & (np.floor(z) == 5)] = False
    keep[pick] = True
    x, y, z = x[keep], y[keep], z[keep]
    w = rng.random(len(x), dtype=np.float32)
    s = synth.System("fullest", x, y, z, w, (0.0, 0.0, 0.0), (32, 32, 32), 1.0, 1.0)
    b = oracle.bin_particles(x, y, z, w, s.origin, s.dims, 1.0, 1.0)
    assert b.max_per_cell == n
    ds = device.DeviceSystem(s)
    ds.bin()
    g = ds.binned()
    assert np.array_equal(g["perm"], b.perm) and np.array_equal(g["offsets"], b.offsets)
    assert np.array_equal(g["counts"], b.counts) and g["max_per_cell"] == n
