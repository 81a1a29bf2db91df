"""The x2 upsampling of the field at the edges of its blocks (64 fine columns,
four pairs of rows), on volumes one voxel thick and, in one axis, longer than a
launch's grid: every operation is one rounded FP32 operation, so the result is
NumPy's bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def source(n):
    s = ((np.arange(2 * n, dtype=np.float32) - np.float32(0.5)) * np.float32(0.5))
    s = np.clip(s, np.float32(0), np.float32(n - 1))
    b = np.floor(s)
    i0 = b.astype(np.int64)
    return i0, np.minimum(i0 + 1, n - 1), (s - b).astype(np.float32)


@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 1, 3), (1, 3, 32), (3, 4, 33), (5, 7, 31),
                                   (9, 16, 65), (1, 262200, 1), (65600, 1, 2)])
def test_upsample_is_exact(shape):
    import torch
    from paper_2603_19371_amd import _lib as L
    u = np.random.default_rng(sum(shape)).standard_normal((3,) + shape).astype(np.float32)
    v, one = u, np.float32(1)
    for axis, n in ((3, shape[2]), (2, shape[1]), (1, shape[0])):
        i0, i1, t = source(n)
        t = t.reshape([-1 if k == axis else 1 for k in range(4)])
        v = (one - t) * np.take(v, i0, axis) + t * np.take(v, i1, axis)
    got = L.upsample_field(torch.from_numpy(u).cuda()).cpu().numpy()
    assert np.array_equal(got, np.float32(2) * v)
