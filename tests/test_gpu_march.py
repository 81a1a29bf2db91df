"""The march of large volumes: two 32 x 8 tiles per block and one barrier per
plane in a stand-alone context, one tile and two barriers in the batch.  Both
sum the same terms in the same order, so a pair's run is the same bit for bit;
on volumes whose last block has one tile or part of one, whose last column is
two voxels wide and whose last chunk is short."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    from paper_2603_19371_amd import _lib
    _lib.lib()
    return _lib


# 280, 280, 288 blocks of two tiles (fewer than the CUs' 256 run single tiles)
ROWS, ODD, CHUNK = (61, 105, 130), (61, 97, 130), (90, 90, 98)


def images(L, shape, seed, bf16):
    import torch
    rng = np.random.default_rng(seed)
    F = rng.random(shape, np.float32)
    M = (0.6 * F + 0.4 * rng.random(shape, np.float32)).astype(np.float32)
    return [torch.from_numpy(v).cuda().to(torch.bfloat16 if bf16 else torch.float32)
            for v in (F, M)]


@pytest.mark.parametrize("accum", [0, 1])
@pytest.mark.parametrize("shape,window,sigma,bf16", [(ROWS, 3, 0.3, False), (ODD, 5, 0.6, True),
                                                     (CHUNK, 7, 1.0, False), (ODD, 7, 1.3, True),
                                                     (ROWS, 9, 1.0, False), (CHUNK, 9, 1.3, True)])
def test_context_and_batch_march_alike(L, shape, window, sigma, bf16, accum):
    import torch
    Ft, Mt = images(L, shape, window, bf16)
    dt = Ft.dtype
    kw = dict(window=window, grad_sigma=sigma, accum=accum, stencil=L.LMR_STENCIL_MARCH)
    ctx = L.Context(shape, img_dtype=dt, **kw)
    ctx.begin(Ft, Mt)
    ctx.step(Ft, Mt, 4)
    batch = L.Batch([shape], img_dtype=dt, **kw)
    batch.begin([Ft], [Mt])
    batch.step(4, graph=True)
    batch.sync()
    pair = batch.pair(0)
    assert ctx.state() == pair.state()
    assert torch.equal(ctx.field(), pair.field())
    assert torch.equal(ctx.grad(), pair.grad())


@pytest.mark.parametrize("sigma", [1.6, 2.0])
def test_widest_gaussians_agree_with_bricks(L, sigma):
    """Radii the batch does not take.  The raw gradients of the two forms agree
    to 2e-5 of max |g| (maps rounded to FP32, whose box sums cancel by two
    digits); the Gaussian (weights of sum 1) keeps that and sums its 13 rounded
    terms per axis in another order: 3 x 13 x 6e-8 more."""
    import torch
    Ft, Mt = images(L, ODD, 11, False)
    u = torch.zeros((3,) + ODD, device="cuda")
    (_, raw, a, _), (_, _, b, _) = [
        L.Context(ODD, window=5, grad_sigma=sigma, stencil=form).loss_grad(Ft, Mt, u)
        for form in (L.LMR_STENCIL_MARCH, L.LMR_STENCIL_CUBE)]
    assert (a - b).abs().max() <= 2.3e-5 * raw.abs().max()
