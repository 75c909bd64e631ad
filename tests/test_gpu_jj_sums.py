"""The per-point sums of vbar and vbar^2 where their reduction (one wavefront
a point over its path chunks) can go wrong: fewer chunks than lanes, exactly
64 and 65 of them, several hundred, and points of different sizes whose last
workgroup is partly empty.

Tolerance: FP64 sums of at most a few hundred thousand terms in another
order than numpy's: 1e-12 relative to the sum of absolute values.
"""
import numpy as np
import pytest
import torch

import sde_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ppt", [1, 2, 4])
@pytest.mark.parametrize("f64", [False, True])
def test_point_sums_over_many_chunks(gpu, ppt, f64):
    sde, ctx, dev = gpu
    sde.sde_set_option(ctx, sde.SDE_OPT_JJ_PPT, ppt)
    paths = [1, 64 * 63, 64 * 64 + 1, 64 * 65, 64 * 300 + 7]
    pts = [sde_inputs.jj_point(n_paths=p, n_steps=8, n_transient=2, f=0.1 * k) for k, p in enumerate(paths)]
    n = sum(paths)
    t = torch.float64 if f64 else torch.float32
    theta, v = torch.zeros(n, dtype=t, device=dev), torch.zeros(n, dtype=t, device=dev)
    wd = torch.zeros(n, dtype=torch.int32, device=dev)
    acc = torch.zeros(n, dtype=torch.float64, device=dev)
    ps = torch.full((len(pts), 2), -1.0, dtype=torch.float64, device=dev)
    run = sde.sde_jj_integrate_f64 if f64 else sde.sde_jj_integrate
    run(ctx, pts, sde.make_run(5, sync=1), theta, wd, v, acc, ps)
    vb = acc.cpu().numpy() / 6
    at = 0
    for q, p in enumerate(paths):
        seg = vb[at:at + p]
        at += p
        got = ps[q].cpu().numpy()
        assert abs(got[0] - seg.sum()) <= 1e-12 * np.abs(seg).sum()
        assert abs(got[1] - (seg ** 2).sum()) <= 1e-12 * (seg ** 2).sum()
