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


def one_tile(n, seed=0):
    """n splats over the one tile of a 16x16 view, many of them at equal
    depths (ordered by id then)."""
    scene = scenes.make_scene(n, seed, -0.2, 0.2, -3.0, 0.3, 0)
    scene["mean"][2, :n] = np.round(scene["mean"][2, :n] * 64) / 64
    return scene, scenes.axis_camera(16, 16, 4.0)


# the sizes a sorting workgroup's registers step through, and the first one
# that is left to the radix sorts
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048,
                               2049, 4096, 4097])
def test_one_list_of_every_sort_size(n):
    require_gpu()
    print(f"one list of {n}", flush=True)
    scene, cams = one_tile(n)
    assert check_lists(scene, cams) == n


@pytest.mark.parametrize("n", [2047, 2048, 2049, 4097])
def test_lists_around_a_chunk_of_gaussians(n):
    require_gpu()
    print(f"lists around a chunk, n {n}", flush=True)
    check_lists(scenes.make_scene(n, 8, -1.0, 1.0, -3.5, 0.5, 0), scenes.arc_cameras(3, 4.0, 97, 65))


@pytest.mark.parametrize("w,h", [(1920, 1080), (2064, 1040)])  # 8,160 and 8,385 tiles
def test_lists_around_the_most_tiles_counted_in_lds(w, h):
    require_gpu()
    print(f"lists of {w}x{h}", flush=True)
    check_lists(scenes.make_scene(3_000, 9, -1.0, 1.0, -3.0, 0.5, 0), scenes.arc_cameras(2, 4.0, w, h),
                "spans")


def crowded(base, cams, n=4_200):
    """The scene with n more splats on one point: a list longer than the
    sorting workgroups hold, which sends the job to the radix sorts."""
    extra = scenes.make_scene(n, 77, -0.001, 0.001, -4.0, 0.3, base["deg"])
    total = base["n"] + n
    out = dict(n=total, deg=base["deg"], ld=scenes.round_up(total))
    for k in ("mean", "log_scale", "quat", "opacity", "sh"):
        out[k] = np.zeros(base[k].shape[:-1] + (out["ld"],), np.float32)
        out[k][..., :base["n"]] = base[k][..., :base["n"]]
        out[k][..., base["n"]:total] = extra[k][..., :n]
    out["quat"][0, total:] = 1.0
    return out, cams


@pytest.mark.parametrize("tileset", ["rect", "spans"])
@pytest.mark.parametrize("views", [1, 4])
def test_lists_of_a_crowded_tile(views, tileset):
    require_gpu()
    print(f"crowded tile, {views} views, {tileset}", flush=True)
    check_lists(*crowded(scenes.make_scene(6_000, 4, -1.0, 1.0, -3.5, 0.5, 0),
                         scenes.arc_cameras(views, 4.0, 150, 100)), tileset)


def test_lists_of_a_crowded_tile_beyond_32_bit_keys():
    """Depths from 3 to 1e9 in 20 views: the view does not fit above the
    depth bits of a 32-bit key."""
    require_gpu()
    print("crowded tile, 64-bit keys", flush=True)
    base = scenes.make_scene(500, 7, -1.0, 1.0, -4.0, 0.5, 0)
    for j, z in enumerate((1e9, 5e8, 2e9)):
        base["mean"][:, j] = (0.0, 0.0, z)
        base["log_scale"][:, j] = np.log(1e6)
        base["opacity"][j] = 3.0
    one = scenes.axis_camera(64, 48, 4.0)
    check_lists(*crowded(base, {k: np.concatenate([v] * 20) for k, v in one.items()}))


@pytest.mark.parametrize("tileset", ["rect", "spans"])
def test_lists_of_a_crowded_tile_with_views_that_see_nothing(tileset):
    require_gpu()
    print(f"crowded tile, empty views, {tileset}", flush=True)
    seen = scenes.arc_cameras(2, 5.0, 96, 64, azimuth_deg=40.0)
    away = {k: v[:1].copy() for k, v in seen.items()}
    away["t"] = away["t"] * -3.0  # the scene lies behind this camera
    order = [away, {k: v[:1] for k, v in seen.items()}, away, away,
             {k: v[1:] for k, v in seen.items()}, away]
    cams = {k: np.concatenate([c[k] for c in order]) for k in seen}
    check_lists(*crowded(scenes.make_scene(3_000, 41, -1.0, 1.0, -4.0, 0.5, 0), cams), tileset)
