"""The FP64 force at phases far from [0, 1), where a diverged path's predictor
or a caller's state may be: the exact sine or cosine of the fraction that the
double holds, as a library function gives it, read off one overdamped Euler
step without noise, whose velocity is the force.  3 ulp (7e-16 relative) as
within [0, 1): the revolutions are taken out exactly.
"""
import numpy as np
import pytest
import torch

import sde_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ppt", [0, 1, 2])
@pytest.mark.parametrize("cosine", [False, True])
def test_force_far_out(gpu, ppt, cosine):
    sde, ctx, dev = gpu
    sde.sde_set_option(ctx, sde.SDE_OPT_JJ_PPT, ppt)
    rng = np.random.default_rng(5)
    theta = np.concatenate([s * 2.0 ** e * rng.uniform(1, 2, 20) for s in (1, -1) for e in range(0, 62)] +
                           [np.array([2.0 ** 42, 2.0 ** 43 + 0.25, -2.0 ** 44 - 0.125, 2.0 ** 51 + 0.5, 1e300, -1e300])])
    n = len(theta)
    pt = sde_inputs.jj_point(n_paths=n, n_steps=1, m=0.0, gamma=1.0, a=0.0, f=0.0, D=0.0,
                             potential=sde_inputs.POT_SIN2PI if cosine else sde_inputs.POT_SIN)
    st = (torch.from_numpy(theta).to(dev), torch.zeros(n, dtype=torch.int32, device=dev),
          torch.zeros(n, dtype=torch.float64, device=dev), torch.zeros(n, dtype=torch.float64, device=dev))
    sde.sde_jj_integrate_f64(ctx, [pt], sde.make_run(1, init=sde.SDE_INIT_FROM_STATE, scheme=sde.SDE_EULER, sync=1), *st)
    v = st[2].cpu().numpy()
    q = np.rint(4 * np.fmod(theta, 1.0))  # exact: fmod is, and the products by 4
    r = (np.fmod(theta, 1.0) - q / 4).astype(np.longdouble) * 2 * np.longdouble("3.14159265358979323846264338327950288")
    k = (q.astype(np.int64) + (1 if cosine else 0)) % 4
    shape = np.choose(k, [np.sin(r), np.cos(r), -np.sin(r), -np.cos(r)])
    ref = -(np.longdouble(2 * np.pi) if cosine else 1) * shape
    assert np.all(np.abs(v - ref) <= 7e-16 * np.abs(ref))
