"""A voxel that is not finite reaches the windows that hold it and no others on
bricks: with compensated box sums, whose z sums run, the same voxels as with
FP64 sums, which are formed one by one."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("window", [3, 5, 7, 9])
@pytest.mark.parametrize("shape", [(24, 30, 41), (67, 83, 71), (196, 37, 61)])
def test_only_the_windows_that_hold_it(shape, window, value):
    import torch
    from paper_2603_19371_amd import _lib as L
    g = torch.Generator(device="cuda")
    g.manual_seed(window)
    F, M = (torch.rand(shape, generator=g, device="cuda") for _ in range(2))
    z, y, x = (s // 2 for s in shape)
    for M_at in [(z, y, x), (z + 1, y - 3, x), (z - 9, 2, x - 7), (z + 6, y + 5, 1)]:
        M[M_at] = value
    u = torch.zeros((3,) + shape, device="cuda")
    lost = []
    for accum in (0, 1):
        ctx = L.Context(shape, window=window, accum=accum, stencil=L.LMR_STENCIL_CUBE)
        lost.append(~torch.isfinite(ctx.loss_grad(F, M, u, smooth=False)[1]))
        ctx.close()
    assert lost[0].any() and not lost[0].all()
    assert torch.equal(*lost)
