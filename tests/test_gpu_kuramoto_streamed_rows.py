"""The streamed mean field where the rows of a slice that LDS holds can go
wrong: one row and less, whole and ragged batches of four rows, slices whose
phases and carry fit (18 rows, 16 of them with the carry), fit without all of
the carry, just fit (36 rows) and reach past it.

One realization per CU, so that a slice is a whole realization; two of them
against the FP64 oracle.  Tolerance: that of the first steps of every mean
field test, 1e-5 max(|phi|, 1) per oscillator and 1e-6 in r.
"""
import numpy as np
import pytest
import torch

import oracle
import sde_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("N", [1, 700, 1024, 1025, 4095, 4097, 16 * 1024, 18 * 1024 - 3, 20 * 1024 + 1, 33 * 1024 + 5,
                               36 * 1024 - 1, 36 * 1024, 36 * 1024 + 1, 43 * 1024 + 17])
def test_streamed_rows(gpu, N, scheme):
    sde, ctx, dev = gpu
    R, steps = torch.cuda.get_device_properties(dev).multi_processor_count, 8
    cfg = sde_inputs.kuramoto_uniform(N=N, R=2)
    ph = torch.empty((R, N), dtype=torch.float32, device=dev)
    rs = torch.zeros((R, 3), dtype=torch.float64, device=dev)
    run = sde.make_run(cfg["seed"], step0=0, scheme=scheme, init=sde.SDE_INIT_PHILOX, sample_every=4, sync=1)
    sde.sde_set_option(ctx, sde.SDE_OPT_KURA_MF, 1)
    try:
        sde.sde_kuramoto_integrate(ctx, sde.sde_kuramoto_desc(N, R, cfg["K"], cfg["D"], cfg["dt"], steps,
                                                              sde.SDE_MEANFIELD, 0), run, ph,
                                   torch.from_numpy(cfg["omega"]).to(dev), None, rs)
    finally:
        sde.sde_set_option(ctx, sde.SDE_OPT_KURA_MF, 0)
    assert sde.sde_get_stats(ctx)["mf_streamed"] == 1
    assert bool(torch.isfinite(ph).all())
    ref, rref = oracle.kuramoto_integrate(N, 2, cfg["K"], cfg["D"], cfg["dt"], steps, 4, oracle.MEANFIELD, scheme,
                                          cfg["seed"], cfg["omega"].astype(np.float64))
    d = 2 * np.pi * ph[:2].cpu().numpy().astype(np.float64) - ref
    d = np.mod(d + np.pi, 2 * np.pi) - np.pi
    assert np.max(np.abs(d) / np.maximum(np.abs(ref), 1.0)) <= 1e-5
    assert np.max(np.abs(rs[:2].cpu().numpy() - rref)) <= 1e-6
