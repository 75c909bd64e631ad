"""sde_observables where its slices can go wrong: groups around the slice
lengths (1024, 2048 and 4096 elements, chosen from the call's total), empty
and single-element groups among them, values far from zero, infinities and
NaN.

Tolerance: every sum is a tree of at most 16 + 8 + 2 + slices/256 + 8
additions deep per element, so its relative error against the sum of the
absolute values stays below 64 ulp of FP64 (1.5e-14) for the slice counts
here; the standard error inherits it through the mean and one square root.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = 1.5e-14


def _counts(total_at_least, slice_):
    c = [0, 1, 2, 255, 256, 257, slice_ - 1, slice_, slice_ + 1, 0, 2 * slice_, 3 * slice_ + 5, 0]
    rest = total_at_least - sum(c)
    return c + ([rest] if rest > 0 else []) + [3, 0]


@pytest.mark.parametrize("total, slice_", [(9000, 1024), (1 << 20, 2048), ((1 << 21) + 777, 4096)])
@pytest.mark.parametrize("kind", ["SDE_OBS_MEAN_F32", "SDE_OBS_MEAN_F64", "SDE_OBS_MEANSQ_F32", "SDE_OBS_ORDER"])
def test_slices_against_numpy(gpu, total, slice_, kind):
    sde, ctx, dev = gpu
    counts = _counts(total, slice_)
    n = sum(counts)
    rng = np.random.default_rng(n)
    dt = np.float64 if kind == "SDE_OBS_MEAN_F64" else np.float32
    x = (rng.random(n) if kind == "SDE_OBS_ORDER" else 5.0 + rng.standard_normal(n)).astype(dt)
    got = sde.sde_observables(ctx, getattr(sde, kind), torch.from_numpy(x).to(dev), counts)
    again = sde.sde_observables(ctx, getattr(sde, kind), torch.from_numpy(x).to(dev), counts)
    assert np.array_equal(got, again)
    at = 0
    for g, c in enumerate(counts):
        part = x[at:at + c].astype(np.float64)
        at += c
        if c == 0:
            assert got[g, 0] == 0.0 and got[g, 1] == 0.0
            continue
        if kind == "SDE_OBS_ORDER":
            z = np.exp(2j * np.pi * part).mean()
            # the sums' error is relative to sum |z_j| = c
            assert abs(got[g, 0] - abs(z)) <= TOL
            assert abs(np.exp(2j * np.pi * got[g, 1]) - z / abs(z)) <= TOL / abs(z) + 1e-15
            continue
        if kind == "SDE_OBS_MEANSQ_F32":
            part = part * part
        mean = part.mean()
        assert abs(got[g, 0] - mean) <= TOL * np.abs(part).mean()
        se = part.std(ddof=1) / np.sqrt(c) if c > 1 else 0.0
        assert abs(got[g, 1] - se) <= TOL * (se + np.abs(part).mean() / np.sqrt(c))


def test_nonfinite_values_stay_in_their_group(gpu):
    sde, ctx, dev = gpu
    counts = [5000, 3000, 5000, 700]
    x = np.full(sum(counts), 2.0, dtype=np.float32)
    x[4999] = np.inf
    x[8000 + 17] = np.nan
    got = sde.sde_observables(ctx, sde.SDE_OBS_MEAN_F32, torch.from_numpy(x).to(dev), counts)
    assert got[0, 0] == np.inf and np.isnan(got[0, 1])
    assert tuple(got[1]) == (2.0, 0.0) and tuple(got[3]) == (2.0, 0.0)
    assert np.isnan(got[2, 0]) and np.isnan(got[2, 1])
