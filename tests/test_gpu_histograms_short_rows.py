"""Histograms of rows of few values and many bins, around the lines where the
copies of a bin, the waves of a workgroup and the way past LDS change: bins
around 64 times the values, copies around a sixteenth of them, work around
2048, 4096 and 16384 values and twice the bins, more rows than a grid has.
Whole numbers, compared exactly with numpy.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _check(gpu, rows, n, bins):
    sde, ctx, dev = gpu
    rng = np.random.default_rng(rows + 7 * n + 11 * bins)
    w = rng.integers(-2, bins + 2, (rows, n)).astype(np.int32)
    w[:, : n // 2] = rng.integers(0, 3, (rows, n // 2))  # half of them in a few bins
    t = rng.random((rows, n)).astype(np.float32)
    t[0, 0] = np.nan
    pos = torch.full((rows, bins + 2), 77, dtype=torch.int64, device=dev)
    phase = torch.full((rows, bins + 1), 77, dtype=torch.int64, device=dev)
    sde.sde_position_histograms(ctx, torch.from_numpy(w).to(dev), 0, bins, pos)
    sde.sde_phase_histograms(ctx, torch.from_numpy(t).to(dev), bins, phase)
    row = np.arange(rows)[:, None]
    ref = np.bincount((row * (bins + 2) + np.clip(w, -1, bins) + 1).ravel().astype(np.int64), minlength=rows * (bins + 2))
    assert np.array_equal(pos.cpu().numpy().ravel(), ref)
    b = np.where(np.isnan(t), bins, np.minimum(np.nan_to_num(t).astype(np.float64) * bins, bins - 1)).astype(np.int64)
    ref = np.bincount((row * (bins + 1) + b).ravel(), minlength=rows * (bins + 1))
    assert np.array_equal(phase.cpu().numpy().ravel(), ref)


@pytest.mark.parametrize("n", [1, 10, 63, 64, 65, 1023, 2049, 8192, 16385, 100000])
@pytest.mark.parametrize("bins", [1, 5, 30, 62, 63, 64, 638, 639, 640, 4030, 7000, 16382, 16383, 16384])
def test_short_rows(gpu, n, bins):
    _check(gpu, 3, n, bins)


@pytest.mark.parametrize("n, bins", [(3, 4), (10, 500), (10, 700)])
def test_more_rows_than_a_grid(gpu, n, bins):
    _check(gpu, 66000, n, bins)
