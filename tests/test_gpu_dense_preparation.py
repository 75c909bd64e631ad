"""The preparation of a dense run at the shapes where it can go wrong: N below,
at and past the eight entries a thread splits and the 32 of a block (with odd
N the rows begin at every 4-byte offset from a 16-byte boundary), and the order
parameter of few and of many oscillators.

Tolerances against the FP64 oracle: the variants' own 1e-5 and 1e-4 rad (a
split product keeps 22 or 16 bits of each term) over ten steps.  r sums FP64 terms of FP32
sines, wrong by 2^-20 at the most: 2e-6.
"""
import numpy as np
import pytest
import torch

import oracle
import sde_inputs

pytestmark = pytest.mark.gpu


def _run(gpu, N, R, coupling, omega, K):
    sde, ctx, dev = gpu
    ph = torch.empty((R, N), dtype=torch.float32, device=dev)
    rs = torch.zeros((R, 3), dtype=torch.float64, device=dev)
    run = sde.make_run(23, step0=0, scheme=0, init=sde.SDE_INIT_PHILOX, sample_every=5, sync=1)
    sde.sde_kuramoto_integrate(ctx, sde.sde_kuramoto_desc(N, R, 4.0, 0.05, 0.005, 10, coupling, 0), run, ph,
                               torch.from_numpy(omega).to(dev), K, rs)
    return ph.cpu().numpy(), rs.cpu().numpy()


@pytest.mark.parametrize("coupling, tol", [(2, 1e-5), (3, 1e-4), (4, 1e-5)])
@pytest.mark.parametrize("N", [1, 2, 7, 8, 9, 31, 32, 40, 63, 129, 261])
def test_ragged_matrix(gpu, coupling, tol, N):
    dev = gpu[2]
    Kmat = sde_inputs.dense_coupling(N, 4.0, 21)
    Kmat[N // 2, 0] *= 3.0      # the largest entry, away from the last
    omega = sde_inputs.kuramoto_omega(N, 0.5, 22)
    ref, rref = oracle.kuramoto_integrate(N, 3, 4.0, 0.05, 0.005, 10, 5, oracle.DENSE, 0, 23,
                                          omega.astype(np.float64), Kmat=Kmat.astype(np.float64))
    ph, rs = _run(gpu, N, 3, coupling, omega, torch.from_numpy(Kmat).to(dev))
    d = np.mod(2 * np.pi * ph.astype(np.float64) - ref + np.pi, 2 * np.pi) - np.pi
    assert np.max(np.abs(d) / np.maximum(np.abs(ref), 1.0)) <= tol
    assert np.max(np.abs(rs - rref)) <= 10 * tol


@pytest.mark.parametrize("N", [1, 5, 1023, 1025, 4095, 4097, 9000])
def test_order_parameter(gpu, N):
    """The sample after the last step is r of the phases that the call returns."""
    omega = sde_inputs.kuramoto_omega(N, 0.5, 22)
    sde, ctx, dev = gpu
    ph = torch.empty((2, N), dtype=torch.float32, device=dev)
    rs = torch.zeros((2, 2), dtype=torch.float64, device=dev)
    run = sde.make_run(5, step0=0, scheme=0, init=sde.SDE_INIT_PHILOX, sample_every=2, sync=1)
    sde.sde_kuramoto_integrate(ctx, sde.sde_kuramoto_desc(N, 2, 3.0, 0.1, 0.01, 2, sde.SDE_TILED, 0), run, ph,
                               torch.from_numpy(omega).to(dev), None, rs)
    r = np.abs(np.mean(np.exp(2j * np.pi * ph.cpu().numpy().astype(np.float64)), axis=1))
    assert np.max(np.abs(rs.cpu().numpy()[:, 1] - r)) <= 2e-6
