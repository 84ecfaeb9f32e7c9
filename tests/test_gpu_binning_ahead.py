"""The tile lists that are filled and sorted before the host has read their
counts: a capacity that is too small by one leaves every buffer as it was,
an exact one is enough, and long and short lists of one launch are both
sorted."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_20943_amd import gs, scenes
from tests.gpu_helpers import gpu_forward, lists_to_numpy, require_gpu

pytestmark = pytest.mark.gpu

OPTIONS = gs.GS_PROJECT_TIGHT_RECT | gs.GS_PROJECT_TILE_SPANS


def crowd(n_middle, n_around, views, w=104, h=88):
    """n_middle splats in one tile's sight, n_around everywhere."""
    a = scenes.make_scene(n_middle, 3, -0.02, 0.02, -5.0, 0.3, 0)
    b = scenes.make_scene(n_around, 4, -1.5, 1.5, -4.0, 0.5, 0)
    n = n_middle + n_around
    out = scenes.make_scene(n, 5, -1.0, 1.0, -4.0, 0.5, 0)
    for k in ("mean", "log_scale", "quat", "opacity", "sh"):
        out[k][..., :n_middle] = a[k][..., :n_middle]
        out[k][..., n_middle:n] = b[k][..., :n_around]
    return out, scenes.arc_cameras(views, 4.0, w, h)


@pytest.mark.parametrize("middle", [900, 1100, 3000])
@pytest.mark.parametrize("views,w,h", [
    (1, 104, 88), (3, 104, 88),
    (1, 512, 512), (1, 528, 512),  # 1,024 tiles: four waves a list, 1,056: one
])
def test_long_and_short_lists(middle, views, w, h):
    require_gpu()
    print(f"long and short lists {middle} {views} {w}x{h}", flush=True)
    scene, cams = crowd(middle, 2_000, views, w, h)
    _, _, _, out = gpu_forward(scene, cams)
    L_or = oracle.bin_sort(oracle.project(scene, cams, "rect"), cams)
    L_g = lists_to_numpy(out["lists"])
    longest = np.diff(L_or["ranges"].astype(np.int64), axis=1).max()
    assert middle < longest <= 4096
    for k in ("keys", "vals", "ranges"):
        np.testing.assert_array_equal(L_g[k], L_or[k], err_msg=k)


@pytest.mark.parametrize("middle", [0, 1100, 5000])  # the last by radix sorts
@pytest.mark.parametrize("short_by", [-1, 0, 1, "all"])
def test_capacity(middle, short_by):
    require_gpu()
    print(f"capacity {middle} {short_by}", flush=True)
    scene, cams = crowd(middle, 1_000, 2)
    g, gc, ctx = gs.Gaussians.from_scene(scene), gs.Cameras(cams), gs.default_context()
    n, V = g.n, 2
    proj = gs.Projected.empty(V, n, g.ld, "cuda")
    proj.options = OPTIONS
    gs.gs_project(ctx, g, gc, proj)
    L_or = oracle.bin_sort(oracle.project(scene, cams, "spans"), cams)
    cap = 0 if short_by == "all" else L_or["count"] - short_by
    nseg = gc.n_segments()
    lists = gs.TileLists(cap + 64, nseg)
    lists.c().capacity = cap  # 64 words behind it must stay as they are
    vals, ranges = lists.vals.fill_(-3), lists.ranges.fill_(-5)
    before = proj.splat.clone()
    ws = torch.empty(gs.bin_sort_workspace_size(V, g.ld, cap, nseg), dtype=torch.uint8,
                     device="cuda")
    if short_by == "all" or short_by > 0:
        with pytest.raises(gs.GsError) as e:
            gs.gs_bin_sort(ctx, proj, gc, lists, ws)
        assert e.value.code == gs.GS_ERR_CAPACITY and lists.count == L_or["count"]
        torch.cuda.synchronize()
        assert (vals == -3).all() and (ranges == -5).all()
        assert torch.equal(proj.splat.view(torch.int32), before.view(torch.int32))
    else:
        gs.gs_bin_sort(ctx, proj, gc, lists, ws)
        torch.cuda.synchronize()
        M = L_or["count"]
        assert lists.count == M and (vals[M:] == -3).all()
        np.testing.assert_array_equal(vals[:M].cpu().numpy().view(np.uint32), L_or["vals"])
        np.testing.assert_array_equal(ranges.cpu().numpy().view(np.uint32).reshape(-1, 2),
                                      L_or["ranges"])


# a wave's share of a tile's column: 1 chunk of 2,048 Gaussians, 16, 17 and 33
@pytest.mark.parametrize("n", [2_000, 16 * 16 * 2048, 16 * 16 * 2048 + 1, 33 * 16 * 2048])
def test_columns_of_many_chunks(n):
    require_gpu()
    print(f"columns of {n} Gaussians", flush=True)
    scene = scenes.make_scene(n, 6, -1.0, 1.0, -6.5, 0.3, 0)
    cams = scenes.arc_cameras(1, 4.0, 1040, 1000)
    _, _, _, out = gpu_forward(scene, cams, capacity=1 << 23, tight_rect=True, tile_spans=True)
    L_or = oracle.bin_sort(oracle.project(scene, cams, "spans"), cams)
    L_g = lists_to_numpy(out["lists"])
    assert L_g["count"] == L_or["count"] > n // 2
    assert np.diff(L_or["ranges"].astype(np.int64), axis=1).max() <= 4096
    for k in ("vals", "ranges"):
        np.testing.assert_array_equal(L_g[k], L_or[k], err_msg=k)
