"""The squared error's launch shapes against FP64."""
import pytest
import torch

from paper_2512_20943_amd import gs
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu


# a block steps 4,096 values; 256 blocks of four steps hold 4,194,304
@pytest.mark.parametrize("count", [1, 3, 4095, 4097, 300_001, 4_194_304, 4_194_309, 9_000_002])
@pytest.mark.parametrize("offset", [0, 1])
def test_squared_error_launch_shapes(count, offset):
    require_gpu()
    print(f"sq_error {count} +{offset}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(count)
    a = torch.rand(count + 4, generator=g, device="cuda")[offset:offset + count]
    b = torch.rand(count + 4, generator=g, device="cuda")[offset:offset + count]
    out = torch.full((1,), 2.5, dtype=torch.float64, device="cuda")
    gs.gs_sq_error(gs.default_context(), a, b, out)
    want = 2.5 + float(((a.double() - b.double()) ** 2).cpu().numpy().sum())
    # non-negative FP64 terms: every order of summation is within depth * eps
    assert abs(float(out.item()) - want) <= 1e-12 * want
