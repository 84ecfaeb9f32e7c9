"""Keep-masks of usage pruning made on the device against the host's stable
ordering."""
import math

import numpy as np
import pytest
import torch

from paper_2512_20943_amd import gs, prune
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu


# partitions of the sort hold 8,192 keys; a launch writes 64 masks
@pytest.mark.parametrize("n, grid, levels", [
    (1, (1, 1), 3), (255, (16, 16), 11), (8191, (91, 91), 11), (8192, (91, 91), 64),
    (8193, (97, 85), 65), (30_001, (175, 174), 130), (30_001, (175, 174), 0)])
@pytest.mark.parametrize("kind", ["ties", "all equal", "high bits"])
def test_usage_masks_equal_the_host_ordering(n, grid, levels, kind):
    require_gpu()
    print(f"usage masks {n} {grid} {levels} {kind}", flush=True)
    rng = np.random.default_rng(n + levels)
    u = {"ties": rng.integers(0, 50, n), "all equal": np.full(n, 7),
         "high bits": rng.integers(0, 2 ** 32, n)}[kind].astype(np.uint32)
    gw, gh = grid
    lv = rng.uniform(0.0, 1.0, levels)
    if levels:
        lv[0], lv[-1] = 0.0, 1.0
    want = prune.usage_keep_masks(u, n, gw, gh, lv)
    drops = [int(math.floor(x * n + 1e-9)) for x in lv]
    masks = torch.full((levels, gh, gw), 9, dtype=torch.uint8, device="cuda")
    usage = torch.from_numpy(u.view(np.int32)).cuda()
    gs.gs_usage_masks(gs.default_context(), usage, n, gw, gh, drops, masks)
    np.testing.assert_array_equal(masks.cpu().numpy(),
                                  np.array(want, np.uint8).reshape(levels, gh, gw))
    np.testing.assert_array_equal(usage.cpu().numpy().view(np.uint32), u)


def test_bad_drop_counts_are_refused():
    require_gpu()
    u = torch.zeros(10, dtype=torch.int32, device="cuda")
    m = torch.empty(1, 4, 4, dtype=torch.uint8, device="cuda")
    for drops, gw in (([-1], 4), ([11], 4), ([1], 2)):
        with pytest.raises(gs.GsError):
            gs.gs_usage_masks(gs.default_context(), u, 10, gw, 4, drops, m)
