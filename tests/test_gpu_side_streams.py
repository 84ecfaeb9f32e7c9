"""Calls on a stream that is not torch's current one: what a call promises at
its return holds for every stream, and scratch that a binding allocates is not
handed out again while the call's kernels use it."""
import math

import numpy as np
import pytest
import torch

from paper_2512_20943_amd import gs
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu


# below and above the size whose chunk counts need a scan
@pytest.mark.parametrize("n", [1, 300_000, 4096 * 1024, 4096 * 1024 + 5])
def test_culled_indices_are_complete_at_return(n):
    require_gpu()
    print(f"cull on a side stream, n={n}", flush=True)
    x = np.random.default_rng(n).normal(size=n).astype(np.float32)
    t = torch.from_numpy(x).cuda()
    idx = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    ws = torch.empty(gs.cull_workspace_size(n), dtype=torch.uint8, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    m = gs.gs_cull_low_opacity(gs.default_context(), t, n, 0.3, idx, workspace=ws, stream=side)
    # nothing of the call is left to do, so another stream may use the scratch
    # and read the indices
    assert side.query()
    ws.fill_(0xFF)
    got = idx.cpu().numpy()
    p = float(np.float32(0.3))
    want = np.nonzero(x.astype(np.float64) >= math.log(p / (1.0 - p)))[0]
    assert m == want.size
    np.testing.assert_array_equal(got[:m], want)
    assert (got[m:] == -7).all()
