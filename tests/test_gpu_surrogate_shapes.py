"""The surrogate's training kernels at the shapes where they can go wrong:
no, one and many hidden layers, widths below, at and past the 16-wide blocks
and the 64-wide tiles, batches below and past the 16 and 32 rows of a
workgroup, the 64-row and k slices and their remainders, batches that change
the rows per workgroup.

Against the FP64 oracle MLP.  Tolerances: an FP32 gradient sums up to 256
products a layer and a batch of up to 1100, each addition to 2^-24 of the
partial sum: below 1e-4 of the vector's norm; the loss curve of a few Adam
steps inherits the gradients' error through steps of lr: 1e-4 relative.
"""
import numpy as np
import pytest
import torch

import oracle.mlp as om

pytestmark = pytest.mark.gpu


def _params(seed, widths):
    rng = np.random.default_rng(seed)
    return [(rng.uniform(-1, 1, (o, i)).astype(np.float32).astype(np.float64) / np.float32(np.sqrt(i)),
             rng.uniform(-0.3, 0.3, o).astype(np.float32).astype(np.float64)) for (o, i), _ in om.param_shapes(widths)]


def _f32(ps):
    return [(W.astype(np.float32).astype(np.float64), b.astype(np.float32).astype(np.float64)) for W, b in ps]


def _rel(a, b):
    return np.linalg.norm(np.asarray(a, np.float64) - b) / max(np.linalg.norm(b), 1e-30)


@pytest.mark.parametrize("widths", [[5, 1], [1, 1, 1], [3, 16, 1], [8, 17, 17, 1], [5, 64, 64, 1], [5, 65, 65, 65, 1],
                                    [2, 100, 100, 1], [5, 250, 250, 1], [4, 32, 32, 32, 32, 32, 32, 32, 1]])
@pytest.mark.parametrize("B", [1, 15, 16, 17, 33, 64, 65, 130, 1100])
def test_gradients(gpu, widths, B):
    sde, ctx, dev = gpu
    members = 5
    s = sde.sde_surrogate_create(ctx, widths, members, 7)
    try:
        ps = _f32(_params(B, widths))
        for m in (0, members - 1):
            sde.sde_surrogate_set_params(s, m, om.pack(ps))
        rng = np.random.default_rng(B + 1)
        X = rng.uniform(-1, 1, (B, widths[0])).astype(np.float32)
        y = rng.standard_normal(B).astype(np.float32)
        ref_loss, ref_g = om.loss_and_grad(ps, X.astype(np.float64), y.astype(np.float64))
        for m in (0, members - 1):
            loss, g = sde.sde_surrogate_loss_grad(s, m, torch.from_numpy(X).to(dev), torch.from_numpy(y).to(dev))
            assert abs(loss - ref_loss) <= 1e-5 * abs(ref_loss)
            off = 0
            for (W, b) in ref_g:
                for part in (W, b):
                    assert _rel(g[off:off + part.size], part.ravel()) <= 1e-4
                    off += part.size
    finally:
        sde.sde_surrogate_destroy(s)


@pytest.mark.parametrize("widths, B", [([5, 1], 40), ([5, 20, 1], 70), ([5, 100, 100, 1], 300),
                                       ([5, 256, 256, 256, 1], 1024)])
def test_loss_curve_of_full_batches(gpu, widths, B):
    """Epochs of one minibatch that holds every sample: the order does not
    matter, and each loss is taken at the weights the step before left."""
    sde, ctx, dev = gpu
    lr, epochs = 2e-3, 6
    s = sde.sde_surrogate_create(ctx, widths, 3, 11)
    try:
        ps = _f32(_params(3, widths))
        for m in range(3):
            sde.sde_surrogate_set_params(s, m, om.pack(ps))
        rng = np.random.default_rng(5)
        X = rng.uniform(-1, 1, (B, 5)).astype(np.float32)
        y = rng.standard_normal(B).astype(np.float32)
        Xt, yt = torch.from_numpy(X).to(dev), torch.from_numpy(y).to(dev)
        # two calls: the Adam state and the weights carry over
        got = np.concatenate([sde.sde_surrogate_train(s, Xt, yt, sde.make_train_opts(k, B, lr=lr)) for k in (4, 2)])
        mom, vel = om.zeros_like(ps), om.zeros_like(ps)
        ref = []
        for t in range(1, epochs + 1):
            loss, g = om.loss_and_grad(ps, X.astype(np.float64), y.astype(np.float64))
            ref.append(loss)
            ps = om.adam_step(ps, g, mom, vel, t, lr=lr)
        np.testing.assert_allclose(got, ref, rtol=1e-4)
    finally:
        sde.sde_surrogate_destroy(s)


@pytest.mark.parametrize("widths", [[5, 65, 65, 65, 1], [5, 250, 250, 1]])
@pytest.mark.parametrize("B", [2448, 2449, 2500, 4100])
def test_gradients_of_large_batches(gpu, widths, B):
    """On either side of the batch from which five members take 32 samples a
    workgroup (on 256 CUs), the last workgroup ragged."""
    test_gradients(gpu, widths, B)
