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
@pytest.mark.parametrize("period", [1, 3, 4, 7, 200])
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
