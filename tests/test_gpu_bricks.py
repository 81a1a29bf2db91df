"""The bricks of small volumes: wide ones (16 x 16 columns, four planes)
against the march over every window, Gaussian and accumulator, on a volume
ragged against the brick in each axis; and a batch of more pairs than a wave
has lanes, whose wide bricks have to reproduce the stand-alone contexts' small
ones bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    from paper_2603_19371_amd import _lib
    _lib.lib()
    return _lib


@pytest.mark.parametrize("accum", [0, 1])
@pytest.mark.parametrize("window,sigma", [(3, 0.3), (5, 0.6), (7, 1.0), (9, 1.3), (5, 1.6),
                                          (7, 2.0)])
def test_wide_bricks_agree_with_the_march(L, window, sigma, accum):
    """Both forms sum the same terms, the box sums in FP64 (or compensated
    FP32) in different orders: relative errors of 729 2^-53 of a sum, 2500
    times that of a variance, so the loss agrees to 1e-9.  The adjoint maps
    round to FP32 (6e-8 of each), and their box sums cancel by two digits:
    2e-5 of max |g|, as against the oracle."""
    import torch
    shape = (37, 83, 101)  # 10 x 6 x 7 wide bricks, each axis cut
    rng = np.random.default_rng(window)
    F = rng.random(shape, np.float32)
    M = (0.6 * F + 0.4 * rng.random(shape, np.float32)).astype(np.float32)
    u = rng.uniform(-1.5, 1.5, (3,) + shape).astype(np.float32)
    Ft, Mt, ut = (torch.from_numpy(v).cuda() for v in (F, M, u))
    got = {}
    for form in (L.LMR_STENCIL_MARCH, L.LMR_STENCIL_CUBE):
        ctx = L.Context(shape, window=window, grad_sigma=sigma, accum=accum, stencil=form)
        got[form] = ctx.loss_grad(Ft, Mt, ut, cc=True)
    a, b = got[L.LMR_STENCIL_MARCH], got[L.LMR_STENCIL_CUBE]
    assert abs(a[0] - b[0]) < 1e-9
    for x, y in zip(a[1:], b[1:]):
        assert (x - y).abs().max() <= 2e-5 * x.abs().max()


def test_batch_of_many_pairs_matches_single_contexts(L):
    import torch
    rng = np.random.default_rng(5)
    shapes = [(8 + i % 5, 9 + (3 * i) % 11, 10 + (7 * i) % 13) for i in range(70)]
    shapes[20], shapes[69] = (33, 17, 40), (16, 32, 48)
    pairs = []
    for sh in shapes:
        F = rng.random(sh, np.float32)
        M = (0.7 * F + 0.3 * rng.random(sh, np.float32)).astype(np.float32)
        pairs.append((torch.from_numpy(F).cuda(), torch.from_numpy(M).cuda()))
    batch = L.Batch(shapes, window=5)
    batch.begin([p[0] for p in pairs], [p[1] for p in pairs])
    batch.step(4, graph=True)
    batch.sync()
    for i in (0, 1, 20, 63, 64, 65, 69):
        ctx = L.Context(shapes[i], window=5)
        ctx.begin(*pairs[i])
        ctx.step(*pairs[i], 4)
        assert ctx.state() == batch.pair(i).state(), i
        assert torch.equal(ctx.field(), batch.pair(i).field()), i
        assert torch.equal(ctx.grad(), batch.pair(i).grad()), i
