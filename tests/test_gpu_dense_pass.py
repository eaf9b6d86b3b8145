"""The dense pass behind a tile sweep: tiles whose halo overflows, or whose few cells
hold more targets than two rounds, alone and in a batch, bit for bit the no-LDS
walk's outputs; and clustered systems at the occupancies where the static rule
picks tiles take no longer than that walk."""
import time

import numpy as np
import pytest

from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu


def _system(n, side, packed, seed):
    """Half of the particles in `packed` cells in a row, the rest uniform, on a 2^-12 lattice."""
    rng = np.random.default_rng(seed)
    q = rng.integers(0, side << 12, (3, n))
    half = np.arange(n) % 2 == 0
    at = rng.integers(0, packed << 12, n)
    q[0] = np.where(half, at, q[0])
    q[1:] = np.where(half, (side // 2 << 12) + (q[1:] & 4095), q[1:])
    x, y, z = (q * 2.0 ** -12).astype(np.float32)
    return synth.System("dense", x, y, z, synth._weights(rng, n), (0.0, 0.0, 0.0), (side,) * 3, 1.0, 1.0)


# targets of the packed cells within a halo of 1408 and past two rounds of 256; past the halo
SYSTEMS = [(1020, 7, 1), (1026, 7, 1), (1300, 8, 2), (6000, 9, 3), (40000, 17, 5)]
OUT = ("rho", "gx", "gy", "gz", "count")


@pytest.mark.parametrize("precision", ["compensated", "plain"])
@pytest.mark.parametrize("tile", [(3, 3, 3), (4, 4, 4), (6, 6, 6), (16, 4, 3)])
def test_dense_tiles_equal_the_no_lds_walk(precision, tile):
    from paper_2406_16091_amd import device

    systems = [_system(n, side, packed, 17 + i) for i, (n, side, packed) in enumerate(SYSTEMS)]
    ref = []
    for s in systems:
        ds = device.DeviceSystem(s)
        ds.bin()
        got = []
        for org in (dict(sweep="nolds"), dict(sweep="subbox", tile=tile)):
            ds.interact(precision=precision, order="original", **org)
            ds.sync()
            got.append((ds.results(), ds.invariants()["pairs"]))
        assert got[0][1] == got[1][1]
        for k in OUT:
            assert np.array_equal(got[0][0][k], got[1][0][k]), (s.n, k)
        ref.append(got[0])
        ds.close()
    db = device.DeviceBatch(systems)
    db.run(precision=precision, sweep="subbox", tile=tile)
    db.sync()
    for s, r, inv, (want, pairs) in zip(systems, db.results(), db.invariants(), ref):
        assert inv["pairs"] == pairs
        for k in OUT:
            assert np.array_equal(r[k], want[k]), (s.n, k)
    db.close()


def _blobs(n, side, count, seed):
    """Nine in ten particles in `count` blobs of a twentieth of the side, the rest uniform."""
    rng = np.random.default_rng(seed)
    centre = rng.random((count, 3)) * side
    p = centre[rng.integers(0, count, n)] + 0.05 * side * rng.standard_normal((n, 3))
    p = np.where(rng.random((n, 1)) < 0.1, rng.random((n, 3)) * side, p)
    p = np.floor(np.clip(p, 0, side - 2.0 ** -10) * 1024) / 1024
    return synth.System("blobs", *(np.ascontiguousarray(p[:, a], np.float32) for a in range(3)), synth._weights(rng, n),
                        (0.0, 0.0, 0.0), (side,) * 3, 1.0, 1.0)


def _best(run):
    import torch
    t = []
    for _ in range(8):
        t0 = time.perf_counter()
        run()
        torch.cuda.synchronize()
        t.append(time.perf_counter() - t0)
    return min(t)


def test_batches_of_clustered_systems_are_no_slower_than_the_no_lds_walk():
    """On the null stream, which runs a batch's launches one after another."""
    from paper_2406_16091_amd import device

    rng = np.random.default_rng(5)
    sizes = [int(1000 * 20 ** rng.random()) for _ in range(16)]
    systems = [_blobs(n, max(3, round((n / rng.uniform(8, 14)) ** (1 / 3))), 8, 40 + i) for i, n in enumerate(sizes)]
    db = device.DeviceBatch(systems)
    time_of, out = {}, {}
    for sweep in ("auto", "nolds"):
        time_of[sweep] = _best(lambda: db.run(sweep=sweep, stream=0))
        db.sync()
        out[sweep] = db.results()
    for a, b in zip(out["auto"], out["nolds"]):
        for k in OUT:
            assert np.array_equal(a[k], b[k]), k
    assert time_of["auto"] < 1.15 * time_of["nolds"], time_of
    db.close()


def test_clustered_systems_are_no_slower_than_the_no_lds_walk():
    from paper_2406_16091_amd import device, pi

    ctx = device.Context(0)  # a context of its own, in static mode
    pi.pi_tuner_mode(ctx.handle, pi.PI_TUNE_STATIC)
    ds = device.DeviceSystem(_blobs(1 << 20, 51, 64, 3), ctx=ctx)
    ds.bin()
    ds.sync()
    auto, walk = (_best(lambda: ds.interact(sweep=sweep)) for sweep in ("auto", "nolds"))
    assert auto < 1.15 * walk, (auto, walk)
    ds.close()
    pi.pi_ctx_destroy(ctx.handle)
