"""The Adam kernel at the edges of its split: one value per thread, with the
last block partly filled, on either side of one block and of 8192 blocks."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_20943_amd import gs
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu

PAD = 300


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("count", [1, 255, 256, 257, 8192 * 256 - 1, 8192 * 256 + 1, 3_000_017])
def test_adam_matches_oracle_at_every_remainder(count, shift):
    require_gpu()
    ctx = gs.default_context()
    rng = np.random.default_rng(count)
    first = rng.uniform(-0.9, 0.9, count).astype(np.float32)
    grad = rng.normal(size=count).astype(np.float32)
    zero = np.zeros(count, np.float32)
    held = [torch.full((shift + count + PAD,), -7.0, device="cuda") for _ in range(4)]
    p, g, m, v = planes = [whole[shift:shift + count] for whole in held]
    for plane, values in zip(planes, (first, grad, zero, zero)):
        plane.copy_(torch.from_numpy(values))
    want, wm, wv = first.astype(np.float64), np.zeros(count), np.zeros(count)
    for step in range(1, 4):
        want, wm, wv = oracle.adam(want, grad, wm, wv, step)
        gs.gs_adam_step(ctx, p, g, m, v, step)
    # p: three roundings of a value below 1 (3e-8 each) and three updates of
    # at most 1e-3 whose second moment holds 1 - 0.999f, 3e-5 off (half of
    # that behind the root); v: the same 3e-5 and its roundings; m: 1 - 0.9f
    # (3e-7) and its roundings; both sums are of terms of one sign, because
    # the gradient stays the same
    np.testing.assert_allclose(p.cpu().numpy(), want, rtol=0, atol=2e-7)
    np.testing.assert_allclose(m.cpu().numpy(), wm, rtol=1e-6, atol=0)
    np.testing.assert_allclose(v.cpu().numpy(), wv, rtol=5e-5, atol=0)
    assert np.array_equal(g.cpu().numpy(), grad)
    for whole in held:
        assert (whole[:shift] == -7).all() and (whole[shift + count:] == -7).all()
