"""The residual's mask counts at texels i < n only: a mask that ends there, at
every remainder of the four texels that a thread takes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_20943_amd import gs, scenes
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 1_020, 1_021, 1_022, 1_023, 1_024])
def test_a_mask_of_n_texels(n):
    require_gpu()
    print(f"mask of {n} texels", flush=True)
    gw, gh = 32, 40
    D, P = scenes.make_delta(n, gw, gh, 5), np.zeros((8, gh, gw), np.float32)
    mask = scenes.prune_mask(D, n, 0.25)
    d_or, amax_or = oracle.residual_delta(D, P, mask, n)
    d, amax = torch.full((8, gh, gw), 7.0, device="cuda"), torch.zeros(8, device="cuda")
    short = torch.from_numpy(mask.reshape(-1)[:n].copy()).cuda()
    gs.gs_residual_delta(gs.default_context(), torch.from_numpy(D).cuda(),
                         torch.from_numpy(P).cuda(), short, n, gw, gh, d, amax)
    np.testing.assert_array_equal(d.cpu().numpy(), d_or)
    np.testing.assert_array_equal(amax.cpu().numpy(), amax_or)
