"""Low-opacity culling at the edges of its chunks and of the sizes whose chunk
counts are added up without a scan, and the plane gather's groups of eight."""
import math

import numpy as np
import pytest
import torch

from paper_2512_20943_amd import gs
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu

CHUNK, SUMMED = 1024, 4096 * 1024


@pytest.mark.parametrize("n", [0, 1, CHUNK - 1, CHUNK, CHUNK + 1, 257 * CHUNK + 3, SUMMED,
                               SUMMED + 1])
@pytest.mark.parametrize("keep", ["none", "all", "some"])
def test_cull_sizes(n, keep):
    require_gpu()
    print(f"cull n={n} {keep}", flush=True)
    x = np.random.default_rng(n).normal(size=n).astype(np.float32)
    x[:] = {"none": -9.0, "all": 9.0}.get(keep, x)
    x[n // 2:n // 2 + 1] = np.nan  # not >= the threshold: dropped
    t = torch.from_numpy(x).cuda()
    idx = torch.full((n + 1,), -7, dtype=torch.int32, device="cuda")
    m = gs.gs_cull_low_opacity(gs.default_context(), t, n, 0.3, idx)
    want = np.nonzero(x.astype(np.float64) >= math.log(float(np.float32(0.3)) /
                                                       (1.0 - float(np.float32(0.3)))))[0]
    assert m == want.size
    np.testing.assert_array_equal(idx[:m].cpu().numpy(), want)
    assert (idx[m:] == -7).all()


@pytest.mark.parametrize("planes", [1, 7, 8, 9, 59])
@pytest.mark.parametrize("m", [1, 255, 257, 1000])
def test_gather_groups(planes, m):
    require_gpu()
    print(f"gather planes={planes} m={m}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(planes + m)
    src = torch.rand(planes, 1024, generator=g, device="cuda")
    idx = torch.randperm(1024, generator=g, device="cuda")[:m].int()
    dst = torch.full((planes, 1088), -1.0, device="cuda")
    gs.gs_gather_planes(gs.default_context(), src, idx, m, dst)
    assert torch.equal(dst[:, :m], src[:, idx.long()])
    assert (dst[:, m:] == -1.0).all()
