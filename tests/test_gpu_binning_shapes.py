"""Tile lists bit-exact against the oracle at the shapes where the binning's
work split changes: ranges long enough that several workgroups share one,
entries around the edges of a workgroup, with packed and unpacked words."""
import numpy as np
import pytest

import oracle
from paper_2512_20943_amd import scenes
from tests.gpu_helpers import gpu_forward, lists_to_numpy, require_gpu

pytestmark = pytest.mark.gpu


def check_lists(scene, cams, tileset="rect", capacity=1 << 22):
    g, gc, r, out = gpu_forward(scene, cams, capacity=capacity, tight_rect=tileset != "rect",
                                tile_spans=tileset == "spans")
    L_or = oracle.bin_sort(oracle.project(scene, cams, tileset), cams)
    L_g = lists_to_numpy(out["lists"])
    assert L_g["count"] == L_or["count"]
    for k in ("keys", "vals", "ranges"):
        np.testing.assert_array_equal(L_g[k], L_or[k], err_msg=k)
    return L_or["count"]


@pytest.mark.parametrize("tileset", ["rect", "spans"])
@pytest.mark.parametrize("n,ld,w,h,views", [
    (700, 704, 1000, 700, 2),      # packed words; hundreds of tiles an entry
    (700, 704, 640, 480, 1),       # one view: no partition table
    (300, 131_072, 4096, 2064, 1),  # ids and tiles too wide to pack
])
def test_lists_of_large_splats(n, ld, w, h, views, tileset):
    require_gpu()
    print(f"large splats: n {n} ld {ld} {w}x{h} x{views} {tileset}", flush=True)
    scene = scenes.make_scene(n, 3, -1.0, 1.0, -1.5, 0.8, 0, ld=ld)
    cams = scenes.arc_cameras(views, 4.0, w, h)
    count = check_lists(scene, cams, tileset)
    assert count > 100 * n  # 256 entries hold more than a shared range's 8,192


@pytest.mark.parametrize("n", [1, 255, 256, 257, 513])
def test_lists_around_a_workgroup_of_entries(n):
    require_gpu()
    print(f"lists at n {n}", flush=True)
    check_lists(scenes.make_scene(n, 5, -0.5, 0.5, -3.0, 0.5, 0), scenes.arc_cameras(3, 4.0, 97, 65))
