"""Invariants around the number of workgroup records that one stage folds: the
no-LDS sweep writes one record per 256 particles, one stage folds 1024."""
import numpy as np
import pytest

from paper_2406_16091_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 256, 257, 1024 * 256, 1024 * 256 + 1])
def test_invariants_equal_the_sums_of_the_outputs(n):
    from paper_2406_16091_amd import device

    s = synth.box_system(n, 64, 21, 10)
    ds = device.DeviceSystem(s)
    ds.bin()
    ds.interact(sweep="nolds", order="original")
    ds.sync()
    r, inv = ds.results(), ds.invariants()
    assert inv["pairs"] == int(r["count"].astype(np.int64).sum())
    # each target's rho is summed in FP64, rounded to FP32 or before that: 2^-24 of
    # every (non-negative) term, doubled
    rho = float(r["rho"].astype(np.float64).sum())
    assert abs(inv["rho_sum"] - rho) <= 2.0 ** -23 * rho
