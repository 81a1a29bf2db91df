"""The tuner takes a cached choice only for what it was timed on: the same
kernels, stencil form and composition."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(20, 37, 70), (32, 32, 32)]


def test_choices_of_other_batches_are_not_taken(tmp_path):
    import torch
    from paper_2603_19371_amd import _lib as L
    images = [[torch.rand(sh, device="cuda") for sh in SHAPES] for _ in range(2)]
    cache = tmp_path / "tune.txt"

    def tune(**kw):
        return L.Batch(SHAPES, window=5, **kw).tune(*images, cache_path=str(cache), iters=1)

    tune()
    key, *cfg, ms = cache.read_text().split()
    assert "|v3|" in key

    def planted(k):
        cache.write_text(" ".join([k, *cfg, "12345.0"]) + "\n")

    planted(key)
    assert tune() == 12345.0
    for kw in (dict(stencil=L.LMR_STENCIL_MARCH), dict(compositive=0)):
        assert tune(**kw) < 12345.0, kw
    # as an earlier build wrote it: its version, with and without the new fields
    head, shapes = key.rsplit("|", 1)
    for old in (key.replace("|v3|", "|v2|"),
                "|".join(head.replace("|v3|", "|v2|").split("|")[:-2] + [shapes])):
        planted(old)
        assert tune() < 12345.0, old
