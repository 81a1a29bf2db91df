"""Mutual information at the sizes where its histogram kernels change shape:
one partly filled block, several blocks that do not fill a group of the fold,
more voxels than one sweep of all blocks, and the smallest and largest
histograms; also images with values that are not numbers."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    from paper_2603_19371_amd import _lib
    _lib.lib()
    return _lib


def _pair(shape, seed):
    rng = np.random.default_rng(seed)
    F = rng.random(shape, np.float32)
    M = (0.5 * F + 0.5 * rng.random(shape, np.float32)).astype(np.float32)
    F[: shape[0] // 2] = 0.0  # a background that shares one bin
    u = rng.uniform(-1.4, 1.4, (3,) + shape).astype(np.float32)
    return F, M, u


# 105 voxels: one block; 20x37x70: 26 blocks, 4 groups, the last of 2;
# 89x90x91: 256 blocks, more than one voxel per thread in some sweeps only
@pytest.mark.parametrize("shape", [(3, 5, 7), (20, 37, 70), (89, 90, 91)])
@pytest.mark.parametrize("bins", [8, 32])
def test_mi_matches_oracle(L, orc, shape, bins):
    import torch
    F, M, u = _pair(shape, 3)
    ctx = L.Context(shape, window=3, similarity=3, mi_bins=bins)
    Ft, Mt, ut = (torch.from_numpy(v).cuda() for v in (F, M, u))
    loss, graw, _, _ = ctx.loss_grad(Ft, Mt, ut, smooth=False)
    rL, rg = orc.mi_loss_grad(F, M, u, bins=bins)
    # loss: Mw rounds at 2^-24 of its size, a bin coordinate is up to `bins`
    # of it and a window's slope is below 1: 32 * 6e-8 per voxel, and the
    # histogram rounds each product at 2^-32
    assert abs(loss - rL) < 4e-6 * max(1.0, abs(rL))
    # gradient: the same coordinate error on products of windows and table
    # entries (log2 of ratios, below 20), and FP32 derivatives
    g = graw.cpu().numpy().astype(np.float64)
    assert np.abs(g - rg).max() < 2e-5 * max(1e-12, np.abs(rg).max())


def test_mi_skips_values_that_are_not_numbers(L):
    """A voxel of F that is not a number has no window: it adds nothing to
    the histogram and its own gradient is 0, the others stay finite."""
    import torch
    F, M, u = _pair((20, 37, 70), 4)
    F[15, 7, 9] = np.nan
    ctx = L.Context(F.shape, window=3, similarity=3, mi_bins=32)
    Ft, Mt, ut = (torch.from_numpy(v).cuda() for v in (F, M, u))
    loss, graw, _, _ = ctx.loss_grad(Ft, Mt, ut, smooth=False)
    assert np.isfinite(loss)
    g = graw.cpu().numpy()
    assert np.isfinite(g).all()
    assert (g[:, 15, 7, 9] == 0).all()
