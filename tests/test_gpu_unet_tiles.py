"""The forms of the convolution that the small networks of the other tests do
not reach, each layer alone against the FP64 oracle with the bounds derived in
test_gpu_unet.py (1e-5 of the sum of |products| per output, 1e-4 for the weight
and bias gradients):

  32 output channels per block, where that gives every compute unit a block:
  half resolution of 80x96x112 (480 tiles), and a quarter of 104x136x144
  (189 tiles x 2, cut along every axis);
  operands streamed from memory, for inputs beyond 32-bit byte offsets (4 GiB;
  here by the channel stride alone): K = 16 with 48 channels, K = 32 with 32."""
import numpy as np
import pytest

import test_gpu_unet as U

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    from paper_2603_19371_amd import _lib
    _lib.lib()
    return _lib


@pytest.mark.parametrize("shape,layers", [((80, 96, 112), (2, 3, 10)),
                                          ((104, 136, 144), (5, 8))])
def test_two_channel_tiles_per_block(L, shape, layers):
    U.test_each_layer_matches_oracle_elementwise(L, shape, layers)


@pytest.mark.parametrize("layer,shape", [(12, (8, 8, 8)), (3, (8, 16, 48))])
def test_streamed_operands(L, layer, shape):
    from oracle import unet
    params, _, _, _ = U.make_case(shape, seed=41)
    net = L.UNet(shape)
    net.set_params(torch.from_numpy(U.flat(params)).cuda())
    ci, co, relu = unet.LAYERS[layer]
    dims = tuple(s >> U.LEVEL[layer] for s in shape)
    n = int(np.prod(dims))
    x = U.bf(np.random.default_rng(42).uniform(-1.0, 1.0, (n, ci)))
    xd = torch.empty((n, -(-2 ** 31 // n) + 7 & ~7), dtype=torch.int16, device="cuda")
    xd[:, :ci] = torch.from_numpy(U._bits(x)).cuda()
    y = net.layer_probe(layer, xd)[0].cpu().numpy().astype(np.float64)
    W, b = params[layer]
    X = x.reshape(dims + (ci,))
    ref = np.maximum(unet.conv(X, W, b), 0.0).reshape(n, co)
    top = unet.conv(np.abs(X), np.abs(W), np.abs(b)).reshape(n, co)
    err = np.abs(y - ref) / np.maximum(top, 1e-30)
    print(f"[unet streamed layer {layer} {dims}] y {err.max():.2e} (of sum |products|)")
    assert err.max() <= 1e-5
