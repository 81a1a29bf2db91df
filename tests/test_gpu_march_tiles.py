"""Blocks of two tiles and of one in the march of a stand-alone context, on
either side of the rule between them: an odd row of tiles with short last
columns, rows and chunks (25 columns of blocks, two tiles each); one row of
tiles, and two rows where two tiles per block would leave CUs a coarser load
(one tile each).  Bit for bit the batch, whose blocks run one tile."""
import pytest

import test_gpu_march as march

pytestmark = pytest.mark.gpu

TWO, ROW, FEW = (157, 70, 130), (140, 7, 1100), (110, 15, 700)


@pytest.fixture(scope="module")
def L():
    from paper_2603_19371_amd import _lib
    _lib.lib()
    return _lib


@pytest.mark.parametrize("accum", [0, 1])
@pytest.mark.parametrize("shape,window,sigma,bf16", [
    (TWO, 3, 1.0, True), (TWO, 5, 0.3, False), (TWO, 7, 1.3, False), (TWO, 9, 0.6, True),
    (ROW, 3, 1.3, False), (ROW, 7, 1.0, True), (FEW, 7, 1.0, False), (FEW, 9, 1.3, True)])
def test_context_and_batch_march_alike(L, shape, window, sigma, bf16, accum):
    march.test_context_and_batch_march_alike(L, shape, window, sigma, bf16, accum)
