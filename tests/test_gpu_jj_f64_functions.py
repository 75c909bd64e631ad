"""The FP64 integrator's table functions where they can go wrong, read off
single Euler steps whose other terms vanish, against 64-bit-mantissa long
double (sines at their zeros and between table points, the noise of 2^20
paths from their own Philox words).

Tolerances: a sine, cosine or root is rounded once after a correction of at
most 1 % of it, the amplitude product and the step round once each: 3 ulp
(7e-16 relative); the noise has two functions and three products, 8 ulp
(1.8e-15) of |g| at the most, plus the sum's rounding in v.
"""
import numpy as np
import pytest
import torch

import oracle
import sde_inputs

pytestmark = pytest.mark.gpu


def _euler_step(gpu, pt, theta, v, seed=1):
    sde, ctx, dev = gpu
    n = len(theta)
    st = (torch.from_numpy(theta).to(dev), torch.zeros(n, dtype=torch.int32, device=dev),
          torch.from_numpy(v).to(dev), torch.zeros(n, dtype=torch.float64, device=dev))
    sde.sde_jj_integrate_f64(ctx, [pt], sde.make_run(seed, init=sde.SDE_INIT_FROM_STATE, scheme=sde.SDE_EULER, sync=1),
                             *st)
    return [x.cpu().numpy() for x in st]


def _shape(theta, cosine):
    """sin or cos of 2 pi theta in long double, the quadrant taken out exactly."""
    q = np.rint(4 * theta)
    r = (theta - q / 4).astype(np.longdouble) * 2 * np.longdouble("3.14159265358979323846264338327950288")
    k = (q.astype(np.int64) + (1 if cosine else 0)) % 4
    return np.choose(k, [np.sin(r), np.cos(r), -np.sin(r), -np.cos(r)])


@pytest.mark.parametrize("ppt", [0, 1, 2])
@pytest.mark.parametrize("cosine", [False, True])
def test_force_shape(gpu, ppt, cosine):
    sde, ctx, dev = gpu
    sde.sde_set_option(ctx, sde.SDE_OPT_JJ_PPT, ppt)
    rng = np.random.default_rng(0)
    k = np.arange(0, 512) / 512.0
    eps = 2.0 ** -np.arange(12, 55)
    theta = np.concatenate([k, np.nextafter(k, 1), np.nextafter(k[1:], 0), rng.random(5000), eps, 1 - eps,
                            0.25 + eps, 0.25 - eps, 0.5 + eps, 0.5 - eps, 0.75 + eps, 0.75 - eps, 2.0 ** -np.arange(60, 300, 20.0)])
    theta = theta[(theta >= 0) & (theta < 1)]
    pt = sde_inputs.jj_point(n_paths=len(theta), n_steps=1, a=0.0, f=0.0, D=0.0, gamma=0.0,
                             potential=sde_inputs.POT_SIN2PI if cosine else sde_inputs.POT_SIN)
    v = _euler_step(gpu, pt, theta, np.zeros(len(theta)))[2]
    dt = 2 * np.pi / (pt["omega"] * pt["steps_per_period"])
    ref = -np.longdouble(dt) * (np.longdouble(2 * np.pi) if cosine else 1) * _shape(theta, cosine)
    nearest = ref.astype(np.float64)  # the smallest theta's step underflows to zero
    assert np.all((np.abs(v - ref) <= 7e-16 * np.abs(ref)) | (v == nearest))


def _philox_words(seed, n):
    """Words of Philox4x32-10 at the counters (0, p, 0, NOISE) of paths p < n."""
    m = np.uint64(0xFFFFFFFF)
    c = [np.zeros(n, np.uint64), np.arange(n, dtype=np.uint64), np.zeros(n, np.uint64), np.zeros(n, np.uint64)]
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & m, (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & m]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def test_noise_of_a_million_paths(gpu):
    sde, ctx, dev = gpu
    n, D = 1 << 20, 50.0
    pt = sde_inputs.jj_point(n_paths=n, n_steps=1, a=0.0, f=0.0, D=D, gamma=1.0)
    v = _euler_step(gpu, pt, np.zeros(n), np.zeros(n), seed=77)[2]
    dt = 2 * np.pi / (pt["omega"] * pt["steps_per_period"])
    sigma = np.sqrt(2 * D * dt)
    x = _philox_words(77, n)
    assert [int(w[5]) for w in x] == oracle.philox(77, [0, 5, 0, 0])
    u1 = ((x[0] >> np.uint64(8)) + np.uint64(1)).astype(np.longdouble) / 2 ** 24
    u2 = (x[1] >> np.uint64(8)).astype(np.float64) / 2 ** 24
    ref = np.longdouble(sigma) * np.sqrt(-2 * np.log(u1)) * _shape(u2, True)
    assert np.max(np.abs(ref)) > 4 * sigma
    assert np.all(np.abs(v - ref) <= 1.8e-15 * np.abs(ref) + 2.3e-16 * np.abs(ref))
    # no noise at all: exactly nothing happens at rest
    quiet = dict(pt, D=0.0, n_paths=1000)
    th, wd, vq, acc = _euler_step(gpu, quiet, np.zeros(1000), np.zeros(1000))
    assert np.all(vq == 0.0) and np.all(th == 0.0)
