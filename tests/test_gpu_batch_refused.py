"""A refused lmr_batch_begin leaves the batch as it was: the pairs before the
bad argument keep their images, also in the table that a later call uploads."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes", [[(9, 17, 20), (12, 16, 24)],
                                    [(40, 64, 420), (12, 16, 24)]])
def test_refused_begin_changes_nothing(shapes):
    import torch
    from paper_2603_19371_amd import _lib as L
    rng = np.random.default_rng(3)
    A, B = ([[torch.from_numpy(rng.random(sh, np.float32)).cuda() for sh in shapes]
             for _ in range(2)] for _ in range(2))
    batches = [L.Batch(shapes, window=5) for _ in range(2)]
    for k, b in enumerate(batches):
        b.begin(*A)
        b.step(2, graph=False)
        if k:
            for lam in ([1.0, -1.0], [1.0, float("nan")]):
                with pytest.raises(L.LmrError):
                    b.begin(*B, lambda0=lam)
        b.set_config(0, 16, -1)
        b.step(2, graph=False)
        b.sync()
    for i in range(len(shapes)):
        p, q = (b.pair(i) for b in batches)
        assert p.state() == q.state(), i
        assert torch.equal(p.field(), q.field()), i
