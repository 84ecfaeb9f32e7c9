"""Calls on a stream that is not torch's current one: what a call promises at
its return holds for every stream, and scratch that a binding allocates is not
handed out again while the call's kernels use it."""
import math

import numpy as np
import pytest
import torch

from paper_2512_20943_amd import gs, prune
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


def busy(stream):
    """Some milliseconds of work on a stream."""
    with torch.cuda.stream(stream):
        a = torch.ones(4096, 4096, device="cuda")
        for _ in range(20):
            a = a @ a * 1e-4
    return a


def trample(nbytes):
    """Allocates on the current stream what a block of nbytes could have left
    to it, and writes over it."""
    keep = [torch.empty(max(nbytes, 1), dtype=torch.uint8, device="cuda").fill_(0xFF)
            for _ in range(4)]
    torch.cuda.current_stream().synchronize()
    return keep


@pytest.mark.parametrize("n, grid", [(255, (16, 16)), (300_000, (548, 548))])
def test_usage_masks_keep_their_scratch(n, grid):
    require_gpu()
    print(f"usage masks on a side stream, n={n}", flush=True)
    gw, gh = grid
    u = np.random.default_rng(n).integers(0, 50, n).astype(np.uint32)
    levels = [0.0, 0.3, 0.5, 1.0]
    usage = torch.from_numpy(u.view(np.int32)).cuda()
    masks = torch.full((len(levels), gh, gw), 9, dtype=torch.uint8, device="cuda")
    size = int(gs.load().gs_usage_masks_workspace_size(n))
    side = torch.cuda.Stream()
    trample(size)  # such a block lies ready in the current stream's pool
    torch.cuda.synchronize()
    work = busy(side)
    gs.gs_usage_masks(gs.default_context(), usage, n, gw, gh, [int(x * n + 1e-9) for x in levels],
                      masks, stream=side)
    trample(size)
    torch.cuda.synchronize()
    want = prune.usage_keep_masks(u, n, gw, gh, levels)
    np.testing.assert_array_equal(masks.cpu().numpy(), np.array(want, np.uint8))
    assert work.shape == (4096, 4096)


def test_cull_takes_scratch_of_its_own_stream():
    """The current stream's memory may still be in use there."""
    require_gpu()
    print("cull's own scratch on a side stream", flush=True)
    n = 300_000
    x = np.random.default_rng(4).normal(size=n).astype(np.float32)
    t = torch.from_numpy(x).cuda()
    idx = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    size = gs.cull_workspace_size(n)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    work = busy(torch.cuda.current_stream())
    # freed here with a write of the current stream still to come
    for _ in range(4):
        torch.empty(size, dtype=torch.uint8, device="cuda").fill_(0xFF)
    m = gs.gs_cull_low_opacity(gs.default_context(), t, n, 0.3, idx, stream=side)
    torch.cuda.synchronize()
    p = float(np.float32(0.3))
    want = np.nonzero(x.astype(np.float64) >= math.log(p / (1.0 - p)))[0]
    assert m == want.size and work.shape == (4096, 4096)
    np.testing.assert_array_equal(idx[:m].cpu().numpy(), want)
