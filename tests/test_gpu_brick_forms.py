"""Deep bricks (8 x 8 x 8): a volume whose last one is cut along every axis and
lacks its upper half (49 small bricks deep), whose box passes at windows 3 and 5
and whose Gaussian at any radius take them.  Against the march with the bounds
derived in test_gpu_bricks.py (loss 1e-9, maps and gradients 2e-5 of their
largest), and in batches, whose own bricks are small or wide, bit for bit; and
the squared error, whose reduction has its own blocks, against FP64."""
import numpy as np
import pytest

import test_gpu_batch_bricks as batches

pytestmark = pytest.mark.gpu

SHAPE = (196, 37, 61)


@pytest.fixture(scope="module")
def L():
    from paper_2603_19371_amd import _lib
    _lib.lib()
    return _lib


def images(seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    F = torch.rand(SHAPE, generator=g, device="cuda")
    M = 0.6 * F + 0.4 * torch.rand(SHAPE, generator=g, device="cuda")
    return F, M, 3.0 * torch.rand((3,) + SHAPE, generator=g, device="cuda") - 1.5


@pytest.mark.parametrize("accum", [0, 1])
@pytest.mark.parametrize("window,sigma", [(3, 0.3), (3, 2.0), (5, 0.6), (5, 1.0), (7, 1.3),
                                          (9, 1.6)])
def test_deep_bricks_agree_with_the_march(L, window, sigma, accum):
    F, M, u = images(window)
    a, b = (L.Context(SHAPE, window=window, grad_sigma=sigma, accum=accum, stencil=form)
            .loss_grad(F, M, u, cc=True) for form in (L.LMR_STENCIL_MARCH, L.LMR_STENCIL_CUBE))
    assert abs(a[0] - b[0]) < 1e-9
    for x, y in zip(a[1:], b[1:]):
        assert (x - y).abs().max() <= 2e-5 * x.abs().max()


@pytest.mark.parametrize("accum,bf16,window", [(0, False, 3), (1, True, 3), (0, True, 5),
                                               (1, False, 5)])
def test_batch_matches_contexts_on_deep_bricks(L, accum, bf16, window):
    batches.test_batch_begins_and_runs_as_single_contexts(
        L, [SHAPE, (7, 19, 30)], accum, bf16, window)


@pytest.mark.parametrize("shape", [(1, 1, 1), (5, 7, 9), (60, 70, 80), (130, 200, 330)])
def test_squared_error(L, shape):
    """FP64 sums of FP64 squares of FP32 differences: 1e-12 of the loss."""
    import torch
    F, M = torch.rand(shape, device="cuda"), torch.rand(shape, device="cuda")
    loss = L.Context(shape, similarity=1).loss_grad(F, M, torch.zeros((3,) + shape,
                                                                      device="cuda"))[0]
    exact = float(((F.double() - M.double()) ** 2).mean())
    assert abs(loss - exact) <= 1e-12 * exact
