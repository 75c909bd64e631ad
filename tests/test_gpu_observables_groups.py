"""Observables of many groups, at the lengths where the launch changes: one
wave (256 elements), one workgroup (1024, 4096, and 8192 with 4 groups per
CU), slices past it, groups of the order parameter of any length where there
are enough; lengths mixed, none, and more groups than fit one dimension of a
grid.  Against 64-bit sums: an FP64 sum of n terms in a tree rounds below
40 x 2^-53 of their absolute sum (1e-14 of the mean's scale), the spread and
the angle twice that.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = 1e-14


def _reference(x, counts, kind, sde):
    out, at = np.zeros((len(counts), 2)), 0
    for g, n in enumerate(counts):
        v = x[at:at + n].astype(np.longdouble)
        at += int(n)
        if n == 0:
            continue
        if kind == sde.SDE_OBS_ORDER:
            z = np.exp(2j * np.pi * v.astype(np.float64)).mean()
            out[g] = abs(z), np.angle(z) / (2 * np.pi)
            continue
        v = v * v if kind == sde.SDE_OBS_MEANSQ_F32 else v
        out[g] = v.mean(), (np.sqrt(np.sum((v - v.mean()) ** 2) / (n - 1) / n) if n > 1 else 0.0)
    return out


def _check(gpu, counts, kind_name):
    sde, ctx, dev = gpu
    kind = getattr(sde, kind_name)
    rng = np.random.default_rng(int(sum(counts)) % 1000)
    x = rng.uniform(0.1, 0.4, int(sum(counts)))  # phases far from incoherent, so that the angle is well defined
    x = x if kind == sde.SDE_OBS_MEAN_F64 else x.astype(np.float32)
    got = sde.sde_observables(ctx, kind, torch.from_numpy(x).to(dev), np.array(counts, dtype=np.uint32))
    ref = _reference(x, counts, kind, sde)
    assert np.max(np.abs(got[:, 0] - ref[:, 0])) <= TOL
    assert np.max(np.abs(got[:, 1] - ref[:, 1])) <= 2 * TOL
    again = sde.sde_observables(ctx, kind, torch.from_numpy(x).to(dev), np.array(counts, dtype=np.uint32))
    assert np.array_equal(got, again)


KINDS = ["SDE_OBS_MEAN_F32", "SDE_OBS_MEAN_F64", "SDE_OBS_MEANSQ_F32", "SDE_OBS_ORDER"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("longest", [1, 63, 64, 65, 255, 256, 257, 1024, 1025, 4096, 4097, 8192, 8193, 20000])
@pytest.mark.parametrize("groups", [3, 1024])
def test_lengths(gpu, kind, longest, groups):
    rng = np.random.default_rng(longest)
    counts = rng.integers(0, min(longest, 3000) + 1, groups)
    counts[[0, groups // 2]] = longest
    counts[-1] = 0
    _check(gpu, counts, kind)


@pytest.mark.parametrize("kind", ["SDE_OBS_MEAN_F32", "SDE_OBS_ORDER"])
def test_equal_long_groups(gpu, kind):
    """As many groups as a grid needs, each longer than a slice."""
    _check(gpu, [9000] * 1100, kind)


def test_more_groups_than_one_grid_dimension(gpu):
    sde, ctx, dev = gpu
    n = (1 << 20) + 77
    x = torch.arange(n, dtype=torch.float32, device=dev)
    got = sde.sde_observables(ctx, sde.SDE_OBS_MEAN_F32, x, np.ones(n, dtype=np.uint32))
    assert np.array_equal(got[:, 0], np.arange(n, dtype=np.float32).astype(np.float64))
    assert np.all(got[:, 1] == 0.0)
