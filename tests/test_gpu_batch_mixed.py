"""The persistent batch kernel where a block goes from a brick of one pair to
a marching tile of the next within a phase (one block per CU: 256 blocks; 420
or 96 + 420 bricks before the tiles): every pair as with one launch per phase,
bit for bit, the gradients (the phases without a sum at their end) included."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("window", [3, 7])
@pytest.mark.parametrize("shapes", [[(40, 48, 56), (40, 64, 420)],
                                    [(16, 32, 48), (40, 48, 56), (40, 64, 420)]])
def test_brick_then_tile_in_one_block(shapes, window):
    import torch
    from paper_2603_19371_amd import _lib as L
    rng = np.random.default_rng(window)
    F = [torch.from_numpy(rng.random(sh, np.float32)).cuda() for sh in shapes]
    M = [0.7 * f + 0.3 * torch.rand_like(f) for f in F]
    got = []
    for blocks in (-1, 1):
        b = L.Batch(shapes, window=window, grad_sigma=1.0)
        b.set_config(0, 16, blocks)
        b.begin(F, M)
        b.step(4, graph=False)
        b.sync()
        got.append(b)
    for i in range(len(shapes)):
        p, q = got[0].pair(i), got[1].pair(i)
        assert p.state() == q.state(), i
        assert torch.equal(p.field(), q.field()), i
        assert torch.equal(p.grad(), q.grad()), i
