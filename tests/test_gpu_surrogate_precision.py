"""Error of the ensemble prediction against 64 bits, at rows of few and of many
weights: no larger than that of a plain FP32 network (an FP32 multiply-add
chain per product, z (1 + erf) / 2 rounded after each operation), formed here
from the same weights.  Rows of few weights show the rounding of the operands
and of the activation, which the roundings of a long sum hide.

Each network's output is one unit of its last hidden layer, so nothing is
added to an activation.  5 % over the FP32 network's error, for the chance in
24 networks of 300 queries: a loss of the operands' last bit is worth 30 % and
more at up to four weights a row, a gain of 8 % and more is expected.
"""
import numpy as np
import pytest
import torch
from scipy.special import erf

import oracle.mlp as om

pytestmark = pytest.mark.gpu


def _network(rng, widths, per_row):
    out = []
    for l, ((o, i), _) in enumerate(om.param_shapes(widths)):
        last = l + 2 == len(widths)
        n = 1 if last else i if l == 0 else min(per_row, i)
        W, b = np.zeros((o, i)), np.zeros(o)
        for r in range(o):
            at = rng.choice(i, n, replace=False)
            sign = rng.choice([-1, 1], n) if n > 1 else 1
            W[r, at] = 1.0 if last else rng.uniform(0.75, 1.5, n) * sign * 1.3 / np.sqrt(n)
        if n > 1:
            b = rng.uniform(-0.1, 0.1, o)
        out.append((W.astype(np.float32).astype(np.float64), b.astype(np.float32).astype(np.float64)))
    return out


def _f32_network(params, X):
    """The same network, every operation rounded to FP32 (a multiply-add once)."""
    f = np.float32
    a = X.astype(f)
    for l, (W, b) in enumerate(params):
        z = np.zeros((len(a), W.shape[0]), f)
        for k in range(W.shape[1]):
            z = (z.astype(np.float64) + a[:, k:k + 1].astype(np.float64) * W[None, :, k]).astype(f)
        z = z + b.astype(f)
        if l + 1 < len(params):
            e = erf((z * f(0.70710678118654752)).astype(np.float64)).astype(f)
            z = f(0.5) * z * (f(1.0) + e)
        a = z
    return a[:, 0]


@pytest.mark.parametrize("widths", [[5, 100, 100, 100, 1], [5, 128, 128, 128, 1], [8, 256, 256, 256, 1]], ids=str)
@pytest.mark.parametrize("per_row", [1, 2, 4, 16, 256])
def test_no_further_off_than_fp32(gpu, widths, per_row):
    sde, ctx, dev = gpu
    rng = np.random.default_rng(17 * per_row + widths[1])
    got_sq = f32_sq = ref_sq = 0.0
    for _ in range(24):
        params = _network(rng, widths, per_row)
        X = rng.uniform(0.5, 2.0, (300, widths[0])).astype(np.float32)
        s = sde.sde_surrogate_create(ctx, widths, 1, 3)
        try:
            sde.sde_surrogate_set_params(s, 0, om.pack(params))
            out = torch.zeros((2, len(X)), device=dev)
            sde.sde_surrogate_predict(s, torch.from_numpy(X).to(dev), out[0], out[1])
            got = out[0].cpu().numpy().astype(np.float64)
        finally:
            sde.sde_surrogate_destroy(s)
        ref = om.forward(params, X.astype(np.float64))[0]
        got_sq += np.sum((got - ref) ** 2)
        f32_sq += np.sum((_f32_network(params, X) - ref) ** 2)
        ref_sq += np.sum(ref ** 2)
    print(f"{widths} {per_row} a row: {np.sqrt(got_sq / ref_sq):.2e}, FP32 {np.sqrt(f32_sq / ref_sq):.2e}")
    assert np.sqrt(got_sq) <= 1.05 * np.sqrt(f32_sq)
