"""Histograms where their kernel can go wrong: rows that start at every
4-byte offset of a 16-byte piece and are shorter than one, bin counts around
each number of LDS copies (32, 16, ..., 1, none), every value in one bin,
first bins at and beyond the ends of int32.  Counts are whole numbers:
compared exactly with numpy."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

I32 = np.iinfo(np.int32)


def _positions(w, x0, nb):
    b = np.clip([int(v) - x0 for v in w.tolist()], -1, nb) + 1
    return np.bincount(b.astype(np.int64), minlength=nb + 2)


@pytest.mark.parametrize("offset", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [0, 1, 2, 3, 4, 5, 7, 8, 19, 2047, 4099])
def test_row_starts_and_lengths(gpu, offset, n):
    sde, ctx, dev = gpu
    rows, pitch, nb = 3, n + 5, 6
    rng = np.random.default_rng(100 * n + offset)
    flat = rng.integers(-3, 9, offset + rows * pitch).astype(np.int32)
    w = torch.from_numpy(flat).to(dev)[offset:].view(rows, pitch)
    pos = torch.full((rows, nb + 2), 77, dtype=torch.int64, device=dev)
    sde.sde_position_histograms(ctx, w, 0, nb, pos, n=n)
    t = torch.from_numpy(rng.random(offset + rows * pitch).astype(np.float32)).to(dev)[offset:].view(rows, pitch)
    ph = torch.full((rows, nb + 1), 77, dtype=torch.int64, device=dev)
    sde.sde_phase_histograms(ctx, t, nb, ph, n=n)
    torch.cuda.synchronize()
    for r in range(rows):
        assert np.array_equal(pos[r].cpu().numpy(), _positions(w[r, :n].cpu().numpy(), 0, nb))
        ref = np.bincount((t[r, :n].cpu().double().numpy() * nb).astype(np.int64), minlength=nb + 1)
        assert np.array_equal(ph[r].cpu().numpy(), ref)


@pytest.mark.parametrize("total", [3, 511, 512, 513, 1024, 1025, 4097, 8193, 16384, 16385])
@pytest.mark.parametrize("spread", [0, 10**6])
def test_bin_counts_and_copies(gpu, total, spread):
    sde, ctx, dev = gpu
    n = 100003
    rng = np.random.default_rng(total)
    nb = total - 2
    w = (nb // 2 + rng.integers(-min(spread, nb), min(spread, nb) + 1, (2, n))).astype(np.int32)
    pos = torch.zeros((2, total), dtype=torch.int64, device=dev)
    sde.sde_position_histograms(ctx, torch.from_numpy(w).to(dev), 0, nb, pos)
    torch.cuda.synchronize()
    for r in range(2):
        assert np.array_equal(pos[r].cpu().numpy(), np.bincount(np.clip(w[r], -1, nb) + 1, minlength=total))


@pytest.mark.parametrize("x0", [0, I32.min, I32.min + 1, I32.max, I32.max - 2, I32.min - 1, I32.min - 3, I32.max + 1,
                                -2**40, 2**40])
def test_first_bins_at_the_ends_of_int32(gpu, x0):
    sde, ctx, dev = gpu
    w = np.array([I32.min, I32.min + 1, I32.min + 2, -1, 0, 1, I32.max - 2, I32.max - 1, I32.max] * 5, dtype=np.int32)
    pos = torch.zeros(7, dtype=torch.int64, device=dev)
    sde.sde_position_histogram(ctx, torch.from_numpy(w).to(dev), x0, 5, pos)
    torch.cuda.synchronize()
    assert np.array_equal(pos.cpu().numpy(), _positions(w, x0, 5))
