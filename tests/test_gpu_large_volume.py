"""Volumes of more than 2^31 / 3 voxels, where an element of a field's third
channel (at 2 N + i) or of the fourth adjoint map has no 32-bit index.

The images and the field are random in the last planes and constant before
them, and the same planes as a volume of their own give the reference.  A
sample point is an integer cell and a fraction, so the warp and the update of
a voxel are the same bits there; the gradients agree to 2e-5 of max |g| (box
sums begin at other planes; maps rounded to FP32, whose sums cancel by two
digits).  Planes within 10 of the cut (window and Gaussian 3 + 3 + 3, warp 1)
are left out.  About 110 GB of device memory."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPE, TAIL, CUT = (930, 1000, 832), 40, 10  # 773,760,000 voxels


def test_last_planes_match_a_volume_of_their_own():
    import torch
    from paper_2603_19371_amd import _lib as L
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    sub = (TAIL,) + SHAPE[1:]

    def image():
        t = torch.zeros(SHAPE, dtype=torch.bfloat16, device="cuda")
        t[-TAIL:] = torch.rand(sub, generator=g, device="cuda").to(torch.bfloat16)
        return t

    F, M = image(), image()
    u = torch.zeros((3,) + SHAPE, device="cuda")
    u[:, -TAIL:] = 2.0 * torch.rand((3,) + sub, generator=g, device="cuda") - 1.0
    Fs, Ms, us = F[-TAIL:].clone(), M[-TAIL:].clone(), u[:, -TAIL:].clone()

    def same(big, small, tol, what):
        a, b = big[..., CUT - TAIL:, :, :], small[..., CUT:, :, :]
        err, top = (a - b).abs().max().item(), b.abs().max().item()
        print(f"[large volume] {what}: {err:.3g} of {top:.3g}", flush=True)
        assert err <= tol * top, what

    for big, small in zip(L.warp(M, u, with_grad=True), L.warp(Ms, us, with_grad=True)):
        same(big, small, 0.0, "warp")
        del big
    kw = dict(img_dtype=torch.bfloat16, window=7, grad_sigma=1.0)
    ctx, ref = L.Context(SHAPE, **kw), L.Context(sub, **kw)
    _, raw, smooth, _ = ctx.loss_grad(F, M, u)
    _, raw_s, smooth_s, _ = ref.loss_grad(Fs, Ms, us)
    same(raw, raw_s, 2e-5, "raw gradient")
    same(smooth, smooth_s, 2e-5, "smoothed gradient")
    del raw
    same(ctx.update(u, smooth, 0.5, 0.1),
         ref.update(us, smooth[:, -TAIL:].contiguous(), 0.5, 0.1), 0.0, "update")
    del smooth
    ctx.begin(F, M)
    ref.begin(Fs, Ms)
    same(ctx.grad(), ref.grad(), 2e-5, "gradient at the identity")
    u.fill_(1.0)
    assert not ctx.field(out=u).any()
    ctx.close()
    ctx = L.Context(SHAPE, tile=2, **kw)
    ref = L.Context(sub, tile=2, **kw)
    u.zero_()
    u[:, -TAIL:] = us
    same(ctx.update(u, u, 0.5, 0.1), ref.update(us, us, 0.5, 0.1), 0.0, "pooled update")


def test_more_bricks_than_a_launch_holds():
    """65535 x 1 x 8192 has 16.8 million small bricks, 8.4 million wide ones of
    512 threads: asked for bricks, it marches."""
    import torch
    from paper_2603_19371_amd import _lib as L
    shape = (65535, 1, 8192)
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    F = torch.rand(shape, generator=g, device="cuda", dtype=torch.bfloat16)
    u = torch.zeros((3,) + shape, device="cuda")
    got = []
    for form in (L.LMR_STENCIL_CUBE, L.LMR_STENCIL_MARCH):
        ctx = L.Context(shape, img_dtype=torch.bfloat16, window=7, stencil=form)
        got.append(ctx.loss_grad(F, F, u, smooth=False))
        ctx.close()
    assert got[0][0] == got[1][0]
    assert torch.equal(got[0][1], got[1][1])
