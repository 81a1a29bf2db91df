"""Batches of pairs on bricks, which begin together: few pairs (small bricks
per phase), more (wide bricks), pairs whose stand-alone contexts keep one
partial sum per wide brick (odd numbers of small bricks in x and y), and a
marching pair between them.  Every pair is its stand-alone run bit for bit
from the begin on, with one launch per phase and in the persistent kernel; and
a second begin starts over, also of a pair whose image pointers changed."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# wide bricks: 6 + 8; 330 (83 columns: 11 small bricks, 6 wide ones) + 6 + march;
# 400 + 6 (partial sums per wide brick with every window; above from window 7 on)
BATCHES = [[(7, 19, 30), (15, 9, 23)], [(41, 75, 83), (7, 19, 30), (40, 64, 420)],
           [(100, 64, 64), (7, 19, 30)]]


@pytest.fixture(scope="module")
def L():
    from paper_2603_19371_amd import _lib
    _lib.lib()
    return _lib


@pytest.mark.parametrize("accum,bf16,window", [(0, False, 3), (0, True, 7), (1, False, 9),
                                               (1, True, 5)])
@pytest.mark.parametrize("shapes", BATCHES)
def test_batch_begins_and_runs_as_single_contexts(L, shapes, accum, bf16, window):
    import torch
    dt = torch.bfloat16 if bf16 else torch.float32
    rng = np.random.default_rng(window)
    images = []
    for k in range(2):
        images.append([])
        for sh in shapes:
            F = rng.random(sh, np.float32)
            M = (0.7 * F + 0.3 * rng.random(sh, np.float32)).astype(np.float32)
            images[k].append([torch.from_numpy(v).cuda().to(dt) for v in (F, M)])
    kw = dict(img_dtype=dt, window=window, grad_sigma=1.0, accum=accum)
    lam = [0.5 + i for i in range(len(shapes))]
    for config in ((0, 16, -1), (0, 16, 0)):
        batch = L.Batch(shapes, **kw)
        batch.set_config(*config)
        for k, n in ((0, 0), (0, 3), (1, 2)):
            batch.begin([p[0] for p in images[k]], [p[1] for p in images[k]], lambda0=lam)
            batch.step(n, graph=False)
            batch.sync()
            for i, sh in enumerate(shapes):
                ctx = L.Context(sh, **kw)
                ctx.begin(*images[k][i], lambda0=lam[i])
                ctx.step(*images[k][i], n)
                pair = batch.pair(i)
                assert ctx.state() == pair.state(), (config, k, n, i)
                assert torch.equal(ctx.field(), pair.field()), (config, k, n, i)
                assert torch.equal(ctx.grad(), pair.grad()), (config, k, n, i)
