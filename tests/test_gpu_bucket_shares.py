"""Binning of few particles that lie in few buckets of cells: a bucket of more than
4096 (16384 of at most 32768 in all) is shared by several workgroups.  Every array bit for bit the oracle's, and no
such system much slower than by the radix passes that one particle more would take."""
import time

import numpy as np
import pytest

import oracle
from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu


def _system(n, dims, parts, seed=0):
    """parts: (fraction of the particles, low corner, extents in cells); the rest uniform."""
    rng = np.random.default_rng(n + sum(dims) + seed)
    q = [rng.integers(0, d << 10, n) for d in dims]
    who = rng.random(n)
    lo = 0.0
    for frac, corner, ext in parts:
        mine = (who >= lo) & (who < lo + frac)
        lo += frac
        for a in range(3):
            q[a][mine] = (corner[a] << 10) + rng.integers(0, ext[a] << 10, int(mine.sum()))
    x, y, z = ((v / 1024).astype(np.float32) for v in q)
    return synth.System("shares", x, y, z, rng.random(n, dtype=np.float32), (0.0, 0.0, 0.0), dims, 1.0, 1.0)


G64, G32, G20 = (64, 64, 64), (32, 32, 32), (128, 128, 64)  # buckets of 2^10, 2^7 and 2^12 cells
CASES = [
    (262144, G64, [(1.0, (0, 0, 9), (64, 64, 1))]),    # a layer: four buckets
    (262144, G64, [(1.0, (0, 0, 63), (64, 16, 1))]),   # one bucket
    (262144, G64, [(1.0, (63, 63, 63), (1, 1, 1))]),   # one cell, the last
    (262144, G64, [(1.0, (8, 0, 0), (8, 1, 1))]),      # eight cells
    (262144, G64, [(0.5, (3, 4, 5), (1, 1, 1))]),      # one full cell among uniform ones
    (262144, G64, [(0.3, (0, 0, 0), (9, 9, 9)), (0.3, (40, 40, 40), (3, 3, 3)), (0.3, (60, 2, 33), (2, 2, 2))]),
    (262144, G20, [(1.0, (0, 64, 63), (128, 32, 1))]),  # one bucket of 2^12 cells: seven wavefronts' counters
    (100000, G20, [(0.9, (5, 5, 5), (2, 1, 1))]),
    (262143, G32, [(1.0, (0, 0, 0), (32, 4, 1))]),
    (200001, G32, [(0.7, (1, 1, 1), (2, 2, 2))]),
    (65537, (31, 33, 29), [(1.0, (30, 32, 28), (1, 1, 1))]),
    (4097, G32, [(1.0, (0, 0, 0), (32, 4, 1))]),        # one over a small bucket
    (8192, G32, [(1.0, (0, 0, 0), (32, 4, 1))]),
    (8193, G32, [(1.0, (0, 0, 0), (1, 1, 1))]),
    (12288, G20, [(1.0, (0, 0, 0), (128, 32, 1))]),
    (12289, G20, [(1.0, (0, 0, 0), (2, 2, 1))]),
    (32768, G32, [(1.0, (0, 0, 0), (32, 4, 1))]),       # two shares of 2^14, and shares of 2^12
    (32768, G20, [(0.6, (127, 127, 63), (1, 1, 1))]),
    (32769, G32, [(1.0, (0, 0, 0), (32, 4, 1))]),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_shared_buckets_equal_the_oracle(case):
    from paper_2406_16091_amd import device

    s = _system(*CASES[case])
    b = oracle.bin_particles(s.x, s.y, s.z, s.w, s.origin, s.dims, 1.0, 1.0)
    ds = device.DeviceSystem(s)
    for _ in range(2):
        ds.bin()
    g = ds.binned()
    for k in ("counts", "offsets", "perm"):
        assert np.array_equal(g[k], getattr(b, k)), k
    assert np.array_equal(g["cell"], b.cell[b.perm])
    for k in ("xs", "ys", "zs", "ws"):
        assert np.array_equal(g[k].view(np.uint32), getattr(b, k).view(np.uint32)), k
    assert g["max_per_cell"] == b.max_per_cell
    ds.close()


def _time(s):
    import torch
    from paper_2406_16091_amd import device

    ds = device.DeviceSystem(s)
    ds.bin()
    torch.cuda.synchronize()
    best = 1.0
    for _ in range(5):
        t0 = time.perf_counter()
        for _ in range(20):
            ds.bin()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) / 20)
    ds.close()
    return best


@pytest.mark.parametrize("dims,part", [(G64, ((0, 0, 9), (64, 64, 1))), (G64, ((0, 0, 9), (64, 16, 1))),
                                       (G64, ((3, 4, 5), (1, 1, 1))), (G64, ((8, 0, 0), (8, 1, 1))),
                                       (G32, ((0, 0, 3), (32, 4, 1)))])
def test_concentrated_systems_are_no_slower_than_by_radix_passes(dims, part):
    buckets, passes = (_time(_system(n, dims, [(1.0, *part)])) for n in (262144, 262145))
    assert buckets < 1.25 * passes, (buckets, passes)
