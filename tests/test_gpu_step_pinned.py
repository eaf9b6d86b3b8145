"""Time steps repeat earlier ones bit for bit: state and sweep outputs after eight
steps of small lattice systems against digests of what the library gave before
its sweeps took matrix cores and FP64 (made with the sources of commit 7a8f66a,
every organisation the same there), in every organisation."""
import hashlib

import numpy as np
import pytest

from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu

# particles, cells a side, blobs, seed, force scale
SYSTEMS = {
    "1ppc": (4000, 16, 0, 31, 0.01),
    "8ppc": (6000, 9, 0, 32, 0.01),
    "blobs": (5000, 14, 5, 33, 2e-4),
}
PINNED = {
    ("1ppc", "compensated"): "0967a52d1dbfbe00932f46a4064b4f0c",
    ("1ppc", "fp64acc"): "6fd0a14c7a417bfb1499553160aa7653",
    ("1ppc", "plain"): "49e43c581ec078d6cafd392ea9a28892",
    ("8ppc", "compensated"): "c09d7e3d2e6dd24f297fe7da2b3c804d",
    ("8ppc", "fp64acc"): "58194cd7c01fbb4e10076e2d98d41b0c",
    ("8ppc", "plain"): "1ad6b1c065accf0cb452ad0f54bfddcd",
    ("blobs", "compensated"): "ea0100796a1f331d14960c356d2e9be3",
    ("blobs", "fp64acc"): "18bc795a82f7d15347c2fbdeb047592d",
    ("blobs", "plain"): "a329fe8827aa0c8e77e8dde7f146b224",
}
ORGANISATIONS = [("auto", (0, 0, 0)), ("nolds", (0, 0, 0)), ("stream", (0, 0, 0)), ("pencil", (30, 1, 1)),
                 ("pencilreg", (4, 4, 2)), ("cell", (4, 1, 1)), ("cell", (2, 16, 1))]
ORGANISATIONS += [("subbox", t) for t in ((6, 6, 6), (7, 7, 5), (8, 8, 3), (16, 4, 3), (4, 4, 4), (4, 4, 2), (5, 5, 4),
                                          (5, 4, 4), (5, 4, 3), (4, 4, 3), (4, 3, 3), (3, 3, 3), (3, 3, 2), (3, 2, 2))]
OUTPUTS = ("x", "y", "z", "vx", "vy", "vz", "rho", "gx", "gy", "gz")


def _system(n, side, blobs, seed):
    """Positions on a 2^-14 cell lattice, uniform or in blobs, and lattice velocities."""
    rng = np.random.default_rng(seed)
    q = rng.integers(0, side << 14, (3, n))
    if blobs:
        c = rng.integers(0, side << 14, (blobs, 3))
        q = np.clip(c[rng.integers(0, blobs, n)].T + (q - (side << 13)) // 8, 0, (side << 14) - 1)
    x, y, z = (q * 2.0 ** -14).astype(np.float32)
    w = (0.5 + rng.integers(0, 1 << 20, n) * 2.0 ** -20).astype(np.float32)
    v = [(rng.integers(-(1 << 10), 1 << 10, n) * 2.0 ** -13).astype(np.float32) for _ in range(3)]
    return synth.System("pinned", x, y, z, w, (0.0, 0.0, 0.0), (side,) * 3, 1.0, 1.0), v


@pytest.mark.parametrize("name,precision", sorted(PINNED))
def test_trajectories_are_those_of_earlier_builds(name, precision):
    from paper_2406_16091_amd import device

    n, side, blobs, seed, kappa = SYSTEMS[name]
    s, v = _system(n, side, blobs, seed)
    for sweep, tile in ORGANISATIONS:
        ds = device.DeviceSystem(s)
        ds.bin()
        ds.set_velocity(*v)
        for _ in range(8):
            ds.step(0.25, kappa, 2.0 ** -14, precision=precision, sweep=sweep, tile=tile)
        ds.sync()
        st = ds.state(forces=True)
        digest = hashlib.sha256(b"".join(np.ascontiguousarray(st[k]).tobytes() for k in OUTPUTS)).hexdigest()
        assert digest[:32] == PINNED[name, precision], (sweep, tile)
        ds.close()
