"""The path integrator's loop over whole 4-step blocks, where its events can
go wrong: folds (sample_every) that end a block, fall inside one or on every
step; a window that starts inside a block, on its edge or after the end;
calls that start and stop between blocks; drive periods shorter than a block.

None of these changes a path: theta, winding and v are compared bit for bit
with the run that has no event inside it.  The window sums are compared with
the FP64 oracle: v differs by a few ulp of |v| <= 4 per step without growth
(the -sin phi points are dissipative), at most 7e-7 a step accumulated over
120 steps and summed over as many: 1e-2.  A step too many or too few in the
window is worth |v|, of order 0.5.
"""
import numpy as np
import pytest
import torch

import oracle
import sde_inputs

pytestmark = pytest.mark.gpu

SUM_TOL = 1e-2


def _run(gpu, pts, step0, M, ppt, scheme=0):
    sde, ctx, dev = gpu
    sde.sde_set_option(ctx, sde.SDE_OPT_JJ_PPT, ppt)
    n = sum(p["n_paths"] for p in pts)
    g = torch.Generator().manual_seed(7)
    st = (torch.rand(n, generator=g).to(dev), torch.zeros(n, dtype=torch.int32, device=dev),
          torch.randn(n, generator=g).to(dev), torch.zeros(n, dtype=torch.float64, device=dev))
    start = tuple(x.cpu().double().numpy() for x in st)
    sde.sde_jj_integrate(ctx, pts, sde.make_run(11, step0=step0, init=sde.SDE_INIT_FROM_STATE, sample_every=M,
                                                scheme=scheme, sync=1), *st)
    return start, [x.cpu() for x in st]


@pytest.mark.parametrize("ppt", [0, 1, 2, 4])
@pytest.mark.parametrize("period", [1, 3, 4, 7, 200, 1016, 1017])
@pytest.mark.parametrize("step0, n_steps", [(0, 120), (8, 3), (5, 1), (6, 117), (3, 64)])
def test_events_do_not_touch_the_paths(gpu, ppt, period, step0, n_steps):
    def pts(tr):
        # a drive of period 7 steps or fewer still has a stable step: omega grows with it
        return [sde_inputs.jj_point(n_paths=p, n_steps=n_steps, n_transient=tr, steps_per_period=period,
                                    omega=4.9 * 400 / period, f=0.1) for p in (70, 300)]

    start, base = _run(gpu, pts(step0 + n_steps + 50), step0, 1000, ppt)
    assert torch.all(base[3] == 0)
    end = step0 + n_steps
    for tr in sorted({0, step0, step0 + 1, step0 + 2, step0 + 4, step0 + n_steps // 2, end - 1, end}):
        ref = oracle.jj_integrate(pts(tr), 11, step0=step0,
                                  state=(2 * np.pi * (start[0] + start[1]), start[2], start[3]))
        for M in (1, 2, 3, 4, 6, 40, 100):
            _, got = _run(gpu, pts(tr), step0, M, ppt)
            for a, b in zip(base[:3], got[:3]):
                assert torch.equal(a, b), (tr, M)
            assert np.max(np.abs(got[3].numpy() - ref["acc"])) <= SUM_TOL, (tr, M)


def _state(n, dev, t):
    g = torch.Generator().manual_seed(3)
    return (torch.rand(n, generator=g).to(t).to(dev), torch.zeros(n, dtype=torch.int32, device=dev),
            torch.randn(n, generator=g).to(t).to(dev), torch.zeros(n, dtype=torch.float64, device=dev))


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("period", [2, 5, 100, 1016, 1017])
@pytest.mark.parametrize("step0, n_steps", [(0, 1), (0, 64), (3, 2), (0, 257), (62, 131), (5, 1000)])
def test_noise_drawn_by_other_waves_is_the_same(gpu, f64, scheme, period, step0, n_steps):
    """The launch for small calls (64 paths a workgroup, the noise drawn ahead
    by other waves through an LDS ring) against the persistent kernel: every
    path bit for bit, both potentials, with and without inertia, items that
    end at different blocks of the ring, one of them empty."""
    sde, _, dev = gpu
    pts = [sde_inputs.jj_point(n_paths=p, n_steps=s, n_transient=step0 + s // 3, steps_per_period=period, m=m,
                               omega=4.9 * 400 / period, potential=pot)
           for p, s, m, pot in [(1, n_steps, 1.0, 0), (64, n_steps, 0.0, 1), (65, max(1, n_steps // 2), 1.0, 1),
                                (200, n_steps, 0.0, 0), (30, 0, 1.0, 0), (100, n_steps, 1.0, 0)]]
    n = sum(p["n_paths"] for p in pts)
    t = torch.float64 if f64 else torch.float32
    call = sde.sde_jj_integrate_f64 if f64 else sde.sde_jj_integrate
    ctx = sde.sde_create(0)
    try:
        sde.sde_set_option(ctx, sde.SDE_OPT_AUTOTUNE, 0)
        outs = []
        for ppt in (1, 0):  # the persistent kernel, and the untuned choice for a call this small
            sde.sde_set_option(ctx, sde.SDE_OPT_JJ_PPT, ppt)
            st = _state(n, dev, t)
            ps = torch.zeros((len(pts), 2), dtype=torch.float64, device=dev)
            call(ctx, pts, sde.make_run(4, step0=step0, init=sde.SDE_INIT_FROM_STATE, scheme=scheme, sync=1), *st, ps)
            outs.append([x.cpu() for x in st] + [ps.cpu()])
        for a, b in zip(*outs):
            assert torch.equal(a, b)
    finally:
        sde.sde_destroy(ctx)


def test_recorded_and_noalloc_small_calls(gpu):
    sde, _, dev = gpu
    pts = [sde_inputs.jj_point(n_paths=130, n_steps=403, n_transient=7), sde_inputs.jj_point(n_paths=64, n_steps=96)]
    n = 194
    ctx = sde.sde_create(0)
    try:
        sde.sde_set_option(ctx, sde.SDE_OPT_AUTOTUNE, 0)
        outs = []
        for ppt in (1, 0):
            sde.sde_set_option(ctx, sde.SDE_OPT_JJ_PPT, ppt)
            st = _state(n, dev, torch.float32)
            run = sde.make_run(4, step0=10, init=sde.SDE_INIT_FROM_STATE, sync=1)
            rec = torch.full((60, n), -99, dtype=torch.int32, device=dev)
            sde.sde_jj_integrate_recorded(ctx, pts, run, 8, rec, *st)
            na = _state(n, dev, torch.float32)
            sde.sde_jj_integrate_noalloc(ctx, pts, run, *na)
            torch.cuda.synchronize()
            for a, b in zip(st, na):
                assert torch.equal(a, b)
            outs.append([x.cpu() for x in st] + [rec.cpu()])
        for a, b in zip(*outs):
            assert torch.equal(a, b)
    finally:
        sde.sde_destroy(ctx)
