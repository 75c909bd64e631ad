"""Records and folds that come as often as every block or every step, between
whole blocks of the path integrator: each record is the winding that a call
ending there leaves, no path depends on them, and the window sums are the
same in the launch for small calls and in the persistent one.  Bit for bit.
"""
import pytest
import torch

import sde_inputs

pytestmark = pytest.mark.gpu


def _call(sde, ctx, dev, pts, run, every=0, rows=0):
    n = sum(p["n_paths"] for p in pts)
    g = torch.Generator().manual_seed(3)
    st = (torch.rand(n, generator=g).to(dev), torch.zeros(n, dtype=torch.int32, device=dev),
          (4 * torch.randn(n, generator=g)).clamp_(-8, 8).to(dev), torch.zeros(n, dtype=torch.float64, device=dev))
    rec = torch.full((max(rows, 1), n), -99, dtype=torch.int32, device=dev)
    if every:
        sde.sde_jj_integrate_recorded(ctx, pts, run, every, rec, *st)
    else:
        sde.sde_jj_integrate(ctx, pts, run, *st)
    return [x.cpu() for x in st], rec.cpu()


@pytest.mark.parametrize("ppt", [0, 1, 4])
@pytest.mark.parametrize("every", [4, 8, 12, 100])
@pytest.mark.parametrize("M", [1, 3, 7, 8, 100])
def test_records(gpu, ppt, every, M):
    sde, _, dev = gpu
    ctx = sde.sde_create(0)
    try:
        sde.sde_set_option(ctx, sde.SDE_OPT_AUTOTUNE, 0)
        sde.sde_set_option(ctx, sde.SDE_OPT_JJ_PPT, ppt)
        step0, steps = 6, 131
        rows = (step0 + steps) // every - step0 // every
        run = sde.make_run(4, step0=step0, init=sde.SDE_INIT_FROM_STATE, sample_every=M, sync=1)
        for period, tr in ((3, 0), (400, 61)):
            def pts(n_steps):
                return [sde_inputs.jj_point(n_paths=p, n_steps=n_steps, n_transient=tr, steps_per_period=period,
                                            omega=4.9 * 400 / period) for p in (70, 130)]
            whole, rec = _call(sde, ctx, dev, pts(steps), run, every, rows)
            plain, _ = _call(sde, ctx, dev, pts(steps), sde.make_run(4, step0=step0, init=sde.SDE_INIT_FROM_STATE,
                                                                     sample_every=1000, sync=1))
            assert all(torch.equal(a, b) for a, b in zip(whole[:3], plain[:3]))
            sde.sde_set_option(ctx, sde.SDE_OPT_JJ_PPT, 1)
            one, _ = _call(sde, ctx, dev, pts(steps), run)
            sde.sde_set_option(ctx, sde.SDE_OPT_JJ_PPT, ppt)
            assert torch.equal(whole[3], one[3])
            for r in range(rows):
                at = (step0 // every + r + 1) * every
                end, _ = _call(sde, ctx, dev, pts(at - step0), run)
                assert torch.equal(rec[r], end[1]), (period, r)
    finally:
        sde.sde_destroy(ctx)
