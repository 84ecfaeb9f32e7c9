"""The D-SSIM kernels' band heights (8, 16, 32 or 64 rows by the size of the
launch): loss and gradient against the oracle at ragged sizes of each, and
the calls in which the loss partials may not lie in the gradient."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_20943_amd import gs, scenes
from tests.gpu_helpers import assert_grad_close, require_gpu

pytestmark = pytest.mark.gpu

LOSS_ATOL = 5e-5  # per-pixel SSIM in FP32, C2 = 9e-4


def call(x, y, grad, lam=0.2):
    H, W = x.shape[-2:]
    planes = x.numel() // (H * W)
    ws = torch.empty(gs.l1_dssim_workspace_size(planes, H, W), dtype=torch.uint8, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    gs.gs_l1_dssim_loss_grad(gs.default_context(), x, y, grad, loss, ws, lam)
    return float(loss.item())


def images(shape, seed):
    img, tgt = scenes.image_pair(shape[0], shape[2], shape[3], seed=seed)
    return img, tgt, torch.from_numpy(img).cuda(), torch.from_numpy(tgt).cuda()


# strips x 64-row bands x planes: up to 300 -> 8 rows, 650 -> 16, 1,600 -> 32
@pytest.mark.parametrize("shape", [
    (1, 3, 7, 129), (1, 3, 8, 127), (1, 3, 17, 40), (1, 3, 65, 128),  # 8
    (1, 3, 709, 1281), (2, 3, 513, 900),                              # 396, 432: 16
    (3, 3, 709, 1281),                                                # 1,188: 32
    (5, 3, 709, 1281),                                                # 1,980: 64
])
def test_every_band_height_matches_the_oracle(shape):
    require_gpu()
    print(f"dssim {shape}", flush=True)
    img, tgt, x, y = images(shape, seed=sum(shape))
    grad = torch.full_like(x, float("nan"))
    loss = call(x, y, grad)
    ref_loss, ref_grad = oracle.l1_dssim(img, tgt, 0.2)
    assert abs(loss - ref_loss) <= LOSS_ATOL
    assert_grad_close(grad.cpu().numpy(), ref_grad, f"dL/dI {shape}")


def test_gradients_that_cannot_hold_the_partials():
    """A gradient at an odd float, and in the image's own place: the same
    values as in a buffer of its own."""
    require_gpu()
    print("dssim gradient placement", flush=True)
    _, _, x, y = images((1, 3, 70, 150), seed=4)
    ref = torch.empty_like(x)
    loss = call(x, y, ref)
    buf = torch.full((x.numel() + 1,), float("nan"), device="cuda")
    odd = buf[1:].view(x.shape)
    assert odd.data_ptr() % 8 == 4
    # the partials are then added in another order, in FP64
    assert abs(call(x, y, odd) - loss) <= 1e-12
    assert torch.equal(odd, ref)
    z = x.clone()
    assert abs(call(z, y, z) - loss) <= 1e-12
    assert torch.equal(z, ref)
