"""The sub-box tiles and the stream at the sizes where their matrix-core candidate
test can go wrong: chunks of 64 staged sources and blocks of 16 targets that are full, hold
one entry or are cut by the end of the staged list; targets beyond one round
of 256; a halo at and over its LDS area; rows of targets far
apart; grids narrower than a tile; a cutoff
below the cell width; cell widths far from 1.  On lattice inputs every
organisation sums the same terms in the same order, so outputs equal the no-LDS
walk's bit for bit; counts equal the oracle's."""
import numpy as np
import pytest

from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = [(6, 6, 6), (7, 7, 5), (8, 8, 3), (16, 4, 3), (4, 4, 4), (4, 4, 2), (5, 5, 4), (5, 4, 4), (5, 4, 3), (4, 4, 3),
          (4, 3, 3), (3, 3, 3), (3, 3, 2), (3, 2, 2)]


def _box(n, dims, scale_log2=0, rc_over_w=1.0, seed=7):
    """n particles uniform in dims cells of width 2^scale_log2 on a 2^-12 cell lattice."""
    rng = np.random.default_rng(seed)
    w = 2.0 ** scale_log2
    x, y, z = ((rng.integers(0, d << 12, n) * (w * 2.0 ** -12)).astype(np.float32) for d in dims)
    return synth.System("box", x, y, z, synth._weights(rng, n), (0.0, 0.0, 0.0), dims, w, w * rc_over_w)


def _dense_row(seed=9):
    """Cells of 0 to 150 particles along X, a run longer than a group of targets."""
    rng = np.random.default_rng(seed)
    per = rng.integers(0, 2, 200) * rng.integers(0, 150, 200)
    per[60:140] = 0
    per[[60, 139]] = 1
    ix = np.repeat(np.arange(200), per)
    x = (ix + rng.integers(0, 1 << 12, ix.size) * 2.0 ** -12).astype(np.float32)
    y, z = ((rng.integers(0, d << 12, ix.size) * 2.0 ** -12).astype(np.float32) for d in (2, 1))
    return synth.System("row", x, y, z, synth._weights(rng, ix.size), (0.0, 0.0, 0.0), (200, 2, 1), 1.0, 1.0)


def _some_weights(s, value):
    """Every 50th weight replaced: only the neighbours of those particles see it."""
    s.w[::50] = value
    return s


SYSTEMS = {
    "one": lambda: _box(1, (3, 3, 3)),
    "two_cells": lambda: _box(17, (2, 1, 1)),
    "block16": lambda: _box(16, (4, 4, 2)),
    "chunk64": lambda: _box(64, (4, 4, 2)),
    "chunk65": lambda: _box(65, (4, 4, 2)),
    "rounds": lambda: _box(769, (5, 5, 4)),
    "dense_row": _dense_row,
    "sparse": lambda: _box(700, (997, 3, 2)),
    "one_cell": lambda: _box(700, (1, 1, 1)),
    "thin": lambda: _box(900, (31, 1, 7)),
    "ragged_2ppc": lambda: _box(9001, (17, 13, 21)),
    "ragged_9ppc": lambda: _box(13000, (11, 13, 10)),
    "short_rc": lambda: _box(12000, (13, 15, 17), rc_over_w=0.5),
    "overflow": lambda: _box(20000, (7, 6, 8)),
    "tiny_cells": lambda: _box(6000, (12, 11, 13), scale_log2=-20),
    # the gradient's inner piece overflows float32 (8 / (pi h^5)), the outer does not
    "overflowing_terms": lambda: _box(2500, (12, 11, 13), scale_log2=-28),
    "infinite_weights": lambda: _some_weights(_box(3000, (12, 11, 13)), np.inf),
    "nan_weights": lambda: _some_weights(_box(3000, (12, 11, 13)), np.nan),
    "huge_cells": lambda: _box(6000, (12, 11, 13), scale_log2=40),
}


@pytest.mark.parametrize("name", sorted(SYSTEMS))
@pytest.mark.parametrize("precision", ["compensated", "plain"])
def test_matrix_core_sweeps_equal_the_no_lds_walk(name, precision):
    import oracle
    from paper_2406_16091_amd import device

    s = SYSTEMS[name]()
    ds = device.DeviceSystem(s)
    ds.bin()
    ds.interact(precision=precision, sweep="nolds", order="original")
    ds.sync()
    ref, pairs = ds.results(), ds.invariants()["pairs"]
    b = oracle.bin_particles(s.x, s.y, s.z, s.w, s.origin, s.dims, s.cell_w, s.rc)
    want = oracle.sweep(s.x, s.y, s.z, s.w, s.dims, s.rc, b).count
    assert np.array_equal(ref["count"].astype(np.int64), want)
    for shape in SHAPES + ["stream"]:
        ds.interact(precision=precision, order="original",
                    **(dict(sweep="subbox", tile=shape) if shape != "stream" else dict(sweep=shape)))
        ds.sync()
        got = ds.results()
        for k in ref:
            assert np.array_equal(got[k], ref[k], equal_nan=k != "count"), (name, shape, k)
        assert ds.invariants()["pairs"] == pairs == int(want.sum())
    ds.close()
