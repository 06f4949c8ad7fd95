"""The sums over a pose's tiles behind losses and pose gradients, at numbers of
tiles around the multiples of the rows that are summed side by side (39 for
the 26 sums of the ZNCC gradient, 64 for the others)."""

import numpy as np
import pytest
import torch

from synth import random_poses

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"


@pytest.mark.parametrize("tiles", [1, 38, 39, 40, 63, 64, 65, 156, 157, 256, 257])
def test_losses_and_gradients_from_any_number_of_tiles(tiles):
    """Against FP64 sums over the rendered image and Jacobian, the same FP32
    pixels: only the FP64 rounding of the sums and one FP32 rounding of each
    result are left; 1e-6 of the result, and for a gradient 1e-6 of its terms'
    largest sum of magnitudes, which bounds its cancellation."""
    import paper_2208_12737_amd as P
    g = torch.Generator(device=DEV).manual_seed(tiles)
    vol = P.Volume(torch.rand((22, 25, 27), device=DEV, generator=g), (1.0, 1.1, 0.9), device=DEV)
    det = P.Detector(13, 16 * tiles - 3, 2.0, 40.0 / tiles)
    poses = torch.from_numpy(random_poses(2, 0.4, 3.0, 120.0, seed=3)).to(DEV, torch.float32)
    img, jac = P.render(vol, poses, det, jacobian=True)
    target = img[1].roll(1, dims=-1).contiguous() + 0.5
    I, J, T = img.double(), jac.double(), target.double()
    npix = img[0].numel()

    mi, mt = I.mean((1, 2), keepdim=True), T.mean()
    si, st = I.std((1, 2), keepdim=True, correction=0), T.std(correction=0)
    ih, th = (I - mi) / si, (T - mt) / st
    z = (ih * th).mean((1, 2), keepdim=True)
    per_pixel = -(th - z * ih) / (npix * si)                # d loss / d I
    loss, grad = P.render_ncc_grad(vol, poses, det, target)
    only = P.render_ncc_loss(vol, poses, det, target)
    np.testing.assert_allclose(loss.cpu(), -z[:, 0, 0].cpu(), rtol=1e-6)
    np.testing.assert_allclose(only.cpu(), -z[:, 0, 0].cpu(), rtol=1e-6)
    _close(grad, per_pixel[..., None] * J)

    l2, l2_grad = P.render_l2(vol, poses, det, target)
    np.testing.assert_allclose(l2.cpu(), ((I - T) ** 2).mean((1, 2)).cpu(), rtol=1e-6)
    _close(l2_grad, 2.0 * (I - T)[..., None] * J / npix)
    up = torch.randn(img.shape, device=DEV, generator=g)
    for got in (P.render_backward(det, jac, up), P.render_backward_retrace(vol, poses, det, up)):
        _close(got, up.double()[..., None] * J)


def _close(got, terms):
    want, size = terms.sum((1, 2)), terms.abs().sum((1, 2))
    assert bool(((got.double() - want).abs() <= 1e-6 * size).all())
