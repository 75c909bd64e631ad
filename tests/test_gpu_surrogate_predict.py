"""The ensemble prediction at the shapes where its kernels can go wrong: the
widths on either side of the line between the two kernels, at the 128 and 256
columns the wide one is built for and just past them, 1 to 7 hidden layers,
few and many features, members and queries at the edges of a wave's 16 and a
workgroup's 64 or 128 queries; features and weights far from one, where the
scales of the wide kernel's operands matter; a query that is no number.

Against the FP64 oracle MLP.  Tolerance: every product carries 2^-22 of itself
at the most and a sum of up to 256 of them 24 to 256 roundings of 2^-24 of
partial sums whose magnitude is a few times the result's; with up to 8 layers
that is below 2e-5 of the norm of the members' outputs, and the members' mean
and spread inherit it in units of that norm.
"""
import numpy as np
import pytest
import torch

import oracle.mlp as om

pytestmark = pytest.mark.gpu
TOL = 2e-5


def _params(rng, widths, weight=1.0):
    return [((weight * rng.uniform(-1, 1, (o, i)) / np.sqrt(i)).astype(np.float32).astype(np.float64),
             rng.uniform(-0.3, 0.3, o).astype(np.float32).astype(np.float64)) for (o, i), _ in om.param_shapes(widths)]


def _predict(sde, ctx, dev, params, widths, X, scaling):
    s = sde.sde_surrogate_create(ctx, widths, len(params), 3)
    try:
        for m, ps in enumerate(params):
            sde.sde_surrogate_set_params(s, m, om.pack(ps))
        sde.sde_surrogate_set_scaling(s, sde.make_scaling(*scaling))
        n = len(X)
        out = torch.full((2, n + 3), 7.5, dtype=torch.float32, device=dev)
        sde.sde_surrogate_predict(s, torch.from_numpy(X).to(dev), out[0, :n], out[1, :n])
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert np.all(got[:, n:] == 7.5)
        return got[0, :n], got[1, :n]
    finally:
        sde.sde_surrogate_destroy(s)


def _check(got, params, X, center, scale, mean, std, times_omega):
    outs = np.stack([om.forward(ps, (X.astype(np.float64) - center) / scale)[0] for ps in params])
    outs = (mean + std * outs) * (X[:, 1].astype(np.float64) if times_omega else 1.0)
    norm = np.sqrt(np.mean(outs ** 2))
    err = got[0] - outs.mean(axis=0)
    assert np.sqrt(np.mean(err ** 2)) <= TOL * norm
    spread = outs.std(axis=0, ddof=1) if len(params) > 1 else np.zeros(len(X))
    assert np.sqrt(np.mean((got[1] - spread) ** 2)) <= 2 * TOL * norm


SHAPES = [([1, 64, 64, 1], 2), ([5, 48, 48, 48, 1], 8), ([5, 65, 65, 1], 1), ([5, 100, 100, 100, 1], 5),
          ([8, 127, 127, 1], 3), ([6, 128, 128, 128, 1], 2), ([3, 129, 129, 1], 8), ([5, 200, 200, 200, 1], 5),
          ([5, 256, 256, 256, 1], 5), ([8, 255, 255, 255, 255, 1], 2), ([5, 256, 1], 3), ([2, 20, 1], 2),
          ([5] + [256] * 7 + [1], 2), ([8] + [80] * 7 + [1], 8)]


@pytest.mark.parametrize("widths, members", SHAPES)
@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 65, 127, 128, 129, 1000])
def test_prediction(gpu, widths, members, n):
    sde, ctx, dev = gpu
    rng = np.random.default_rng(n + 7 * len(widths))
    params = [_params(rng, widths) for _ in range(members)]
    X = rng.uniform(1.0, 5.0, (n, widths[0])).astype(np.float32)
    center, scale = [3.0] * widths[0], [2.0] * widths[0]
    times_omega = widths[0] > 1
    got = _predict(sde, ctx, dev, params, widths, X, (center, scale, 0.3, 1.7, times_omega))
    _check(got, params, X, center, scale, 0.3, 1.7, times_omega)


@pytest.mark.parametrize("size", [1e-12, 1e-4, 1e4, 1e12])
@pytest.mark.parametrize("widths", [[5, 100, 100, 1], [5, 256, 256, 256, 1]])
def test_scales(gpu, widths, size):
    """Features far from one, alone and each other's, and members whose
    weights differ by three orders of magnitude."""
    sde, ctx, dev = gpu
    rng = np.random.default_rng(5)
    params = [_params(rng, widths, weight) for weight in (0.03, 1.0, 30.0)]
    X = (rng.uniform(-1.0, 1.0, (300, 5)) * size ** rng.uniform(0.0, 1.0, (300, 1))).astype(np.float32)
    center, scale = [0.0] * 5, [1.0] * 5
    for ps in params:  # the members one by one: their outputs differ as much as their weights
        for i in range(0, 300, 100):  # and by size, so that the largest do not hide the others
            part = X[np.argsort(np.abs(X).max(axis=1))[i:i + 100]]
            got = _predict(sde, ctx, dev, [ps], widths, part, (center, scale, 0.0, 1.0, 0))
            _check(got, [ps], part, np.array(center), np.array(scale), 0.0, 1.0, False)


@pytest.mark.parametrize("widths", [[5, 64, 64, 1], [5, 100, 100, 1], [5, 256, 256, 256, 1]])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_query_that_is_no_number(gpu, widths, bad):
    """It stays no number, and no other query notices."""
    sde, ctx, dev = gpu
    rng = np.random.default_rng(9)
    params = [_params(rng, widths) for _ in range(2)]
    X = rng.uniform(-1.0, 1.0, (200, 5)).astype(np.float32)
    scaling = ([0.0] * 5, [1.0] * 5, 0.0, 1.0, 0)
    clean = _predict(sde, ctx, dev, params, widths, X, scaling)
    X[[3, 16, 150], 2] = bad
    got = _predict(sde, ctx, dev, params, widths, X, scaling)
    for a, b in zip(got, clean):
        assert np.all(np.isnan(a[[3, 16, 150]]))
        keep = np.ones(200, bool)
        keep[[3, 16, 150]] = False
        assert np.array_equal(a[keep], b[keep])


@pytest.mark.parametrize("widths, members", [([5, 70, 70, 1], 5), ([5, 256, 256, 1], 3), ([6, 129, 129, 1], 8),
                                             ([5, 80, 80, 1], 1), ([5, 80, 80, 1], 2),
                                             ([5, 64, 64, 1], 5), ([5, 17, 17, 1], 8), ([5, 250, 1], 3)])
def test_members_in_workgroups_of_their_own(gpu, widths, members):
    """Few workgroups, alone or past the last full round over the CUs, take a
    member each: the same bits as where a workgroup takes them all."""
    sde, ctx, dev = gpu
    rng = np.random.default_rng(2)
    params = [_params(rng, widths) for _ in range(members)]
    per_round = 128 * torch.cuda.get_device_properties(dev).multi_processor_count
    X = rng.uniform(1.0, 5.0, (per_round + 128 * 60 + 3, widths[0])).astype(np.float32)
    scaling = ([3.0] * widths[0], [2.0] * widths[0], 0.3, 1.7, 1)
    whole = _predict(sde, ctx, dev, params, widths, X[:per_round], scaling)
    _check([w[-2000:] for w in whole], params, X[per_round - 2000:per_round], *[np.array(v) for v in scaling[:2]], 0.3, 1.7,
           True)
    for n in (1, 127, 128, 129, 128 * 25 + 1, 128 * 51, 128 * 64 + 5, 128 * 128, 128 * 128 + 1, 128 * 129,
              per_round - 128):
        part = _predict(sde, ctx, dev, params, widths, X[:n], scaling)
        assert all(np.array_equal(p, w[:n]) for p, w in zip(part, whole)), n
    last = _predict(sde, ctx, dev, params, widths, X[-per_round:], scaling)
    for n in (per_round + 1, per_round + 128 * 32, len(X)):
        more = _predict(sde, ctx, dev, params, widths, X[:n], scaling)
        assert all(np.array_equal(m[:per_round], w) for m, w in zip(more, whole)), n
        at = len(X) - per_round
        assert all(np.array_equal(m[at:], e[:n - at]) for m, e in zip(more, last)), n
