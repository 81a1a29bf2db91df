"""The convolutions read their input in 16-byte items where its channel stride
allows, in 8-byte quads otherwise: both give the same bits, at sizes whose
tiles are cut in every direction."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    from paper_2603_19371_amd import _lib
    _lib.lib()
    return _lib


@pytest.mark.parametrize("shape", [(8, 8, 8), (24, 40, 56)])
@pytest.mark.parametrize("layer,level", [(1, 0), (3, 1), (8, 2), (7, 3), (12, 0)])
def test_quad_and_wide_staging_agree(L, shape, layer, level):
    import torch
    from paper_2603_19371_amd import learned
    net = L.UNet(shape)
    net.set_params(torch.from_numpy(learned.init_params(2)).cuda())
    ci, co, _, _ = L.unet_layers()[layer]
    n = int(np.prod([s >> level for s in shape]))
    g = torch.Generator(device="cuda")
    g.manual_seed(layer)
    x = torch.randn(n, ci, generator=g, device="cuda").to(torch.bfloat16)
    dz = torch.randn(n, co, generator=g, device="cuda").to(torch.bfloat16)

    def padded(t, ld):  # the same channels at another stride; the rest is not read
        out = torch.full((n, ld), 3.0, device="cuda").to(torch.bfloat16)
        out[:, :t.shape[1]] = t
        return out.contiguous().view(torch.int16)

    wide = net.layer_probe(layer, padded(x, ci + 8), padded(dz, co + 8))
    quad = net.layer_probe(layer, padded(x, ci + 4), padded(dz, co + 4))
    for a, b, name in zip(wide, quad, ("y", "dx", "dW", "db")):
        assert torch.equal(a, b), name
