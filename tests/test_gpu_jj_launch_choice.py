"""Which launch the path integrator's calls take: shape classes of the tuner on
either side of the limit of the launch for small calls (6 workgroups of 64
paths per CU, FP64 3), which lies inside a power of two of paths.
"""
import pytest
import torch

import sde_inputs

pytestmark = pytest.mark.gpu


def _limit(dev, f64):
    return (3 if f64 else 6) * 64 * torch.cuda.get_device_properties(dev).multi_processor_count


def _integrate(sde, ctx, dev, n_paths, f64, steps=16, period=400):
    pts = [sde_inputs.jj_point(n_paths=n_paths, n_steps=steps, steps_per_period=period, omega=4.9 * 400 / period)]
    ps = torch.zeros((1, 2), dtype=torch.float64, device=dev)
    call = sde.sde_jj_integrate_f64 if f64 else sde.sde_jj_integrate
    call(ctx, pts, sde.make_run(3, sync=1), None, None, None, None, ps)
    return sde.sde_get_stats(ctx)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("first", ["below", "above"])
def test_classes_end_at_the_limit(gpu, f64, first):
    """A call past the limit is tuned for itself, whichever came first."""
    sde, _, dev = gpu
    limit = _limit(dev, f64)
    sizes = [limit, limit + 1] if first == "below" else [limit + 1, limit]
    assert limit.bit_length() == (limit + 1).bit_length()
    ctx = sde.sde_create(0)
    try:
        for n in sizes:
            assert _integrate(sde, ctx, dev, n, f64)["tuned"] == 1
        for n in sizes:
            assert _integrate(sde, ctx, dev, n, f64)["tuned"] == 0
    finally:
        sde.sde_destroy(ctx)


def test_periods_past_the_drive_table_are_a_class(gpu):
    sde, _, dev = gpu
    ctx = sde.sde_create(0)
    try:
        assert [_integrate(sde, ctx, dev, 5000, False, period=p)["tuned"] for p in (1016, 1017, 400, 2000)] == [1, 1, 0, 0]
    finally:
        sde.sde_destroy(ctx)


def _kernels(sde, ctx, dev, n_paths, f64, call=None):
    """Names of the integration kernels that a call launches, as traced."""
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
        if call:
            call()
        else:
            _integrate(sde, ctx, dev, n_paths, f64)
        torch.cuda.synchronize()
    return {k for e in p.key_averages() for k in ("jj_split_kernel", "jj_persistent_kernel") if k in e.key}


@pytest.mark.parametrize("f64", [False, True])
def test_kernel_of_small_and_large_calls(gpu, f64):
    """Untuned calls up to the limit run the split kernel, larger ones and
    forced paths per lane the persistent one: comparisons of the two kernels
    elsewhere rely on it."""
    sde, _, dev = gpu
    limit = _limit(dev, f64)
    ctx = sde.sde_create(0)
    try:
        sde.sde_set_option(ctx, sde.SDE_OPT_AUTOTUNE, 0)
        sde.sde_set_option(ctx, sde.SDE_OPT_GRAPHS, 0)
        assert _kernels(sde, ctx, dev, 1, f64) == {"jj_split_kernel"}
        assert _kernels(sde, ctx, dev, limit, f64) == {"jj_split_kernel"}
        assert _kernels(sde, ctx, dev, limit + 1, f64) == {"jj_persistent_kernel"}
        if not f64:
            pts = [sde_inputs.jj_point(n_paths=194, n_steps=16)]
            assert _kernels(sde, ctx, dev, 0, f64, lambda: sde.sde_jj_integrate_noalloc(
                ctx, pts, sde.make_run(3, sync=1))) == {"jj_split_kernel"}
        for ppt in (1, 2, 4):
            sde.sde_set_option(ctx, sde.SDE_OPT_JJ_PPT, ppt)
            assert _kernels(sde, ctx, dev, 1000, f64) == {"jj_persistent_kernel"}
    finally:
        sde.sde_destroy(ctx)


@pytest.mark.parametrize("cached", [1, 2, 4])
def test_no_allocation_keeps_a_cached_choice_of_fewer_chunks(gpu, tmp_path, cached):
    """A call too large for the scratch is refused with the chunks of the
    choice it would run: 4 paths per lane stay (2 would need twice the
    scratch), 1 falls back to 2, which needs half."""
    sde, _, dev = gpu
    n = 200_000_000
    arch = torch.cuda.get_device_properties(dev).gcnArchName
    key = f"jj|{arch}|f32|scheme0|kinds1|paths2^{n.bit_length() - 1}|steps2^4"
    (tmp_path / "tune.json").write_text('{"%s": %d}' % (key, cached))
    ctx = sde.sde_create(0)
    try:
        sde.sde_set_tune_cache(ctx, str(tmp_path / "tune.json"))
        with pytest.raises(sde.SDEError, match=f"in {-(-n // (64 * max(cached, 2)))} path chunks") as e:
            sde.sde_jj_integrate_noalloc(ctx, [sde_inputs.jj_point(n_paths=n, n_steps=16)], sde.make_run(3, sync=1))
        assert e.value.status == sde.SDE_ERR_INVALID
    finally:
        sde.sde_destroy(ctx)
