"""Kernels and orders of tiles that are chosen by the lists' mean length and the
tiles a splat covers: the same views on both sides of those rules."""
import numpy as np
import pytest
import torch

from paper_2512_20943_amd import gs, scenes
from paper_2512_20943_amd.raster import Rasterizer
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu

W, H = 170, 165  # 121 tiles a view
BG = (0.3, 0.1, 0.2)


def raster():
    return Rasterizer(ctx=gs.Context(torch.cuda.current_device()), capacity=1 << 20,
                      tight_rect=True, tile_spans=True)


def shape(lists, cams, n):
    return lists.count / cams.n_segments(), lists.count / (n * cams.V)


def test_rows_of_ordered_and_unordered_tiles():
    """One wave per tile in launches of 3,630 tiles, longest lists first, and of
    36,300, in launch order: the same row per instance, bit for bit.  (Both are
    binned directly, so rows follow in the order of views and Gaussians; the
    sums over a pair's rows are grouped by the pair's place in its launch.)"""
    require_gpu()
    print("ordered and unordered tiles", flush=True)
    n, small, large = 3_000, 30, 300
    g = gs.Gaussians.from_scene(scenes.make_scene(n, 11, -2.0, 2.0, -2.8, 0.6, 1))
    cams, r = gs.Cameras(scenes.arc_cameras(large, 5.0, W, H)), raster()
    d = torch.rand(large, 3, H, W, generator=torch.Generator("cuda").manual_seed(2), device="cuda")

    def grads(c, dimg):
        out = r.forward(g, c, BG)
        mean, spread = shape(out["lists"], c, n)
        assert 20 <= mean <= 600 and spread <= 30
        grad = gs.Gaussians.zeros_like(g)
        ws = r.backward(g, c, out, dimg, grad, BG)
        rows = ws[c.V * g.ld * 48:][: 36 * out["lists"].count].view(torch.int32).view(-1, 9)
        return rows.clone(), out["proj"].tiles_touched[:, :n].sum(1).cumsum(0).tolist()

    whole, ends = grads(cams, d)
    for v in (0, 90, 270):
        part, part_ends = grads(cams.slice(v, small), d[v:v + small].contiguous())
        first = ends[v - 1] if v else 0
        assert part.abs().max() > 0 and part_ends[-1] == part.shape[0]
        assert torch.equal(part, whole[first:ends[v + small - 1]]), f"views from {v}"


@pytest.mark.parametrize("kind", ["short lists", "wide splats"])
def test_forwards_of_the_two_kernels(kind):
    """Launches of up to 4,000 tiles run one wave per quadrant; larger ones with
    short lists, and ones above 12,000 of wide splats, one per tile."""
    require_gpu()
    print(f"forwards, {kind}", flush=True)
    if kind == "short lists":
        n, mu, large = 200, -3.0, 60
    else:
        n, mu, large = 400, -0.7, 110
    g = gs.Gaussians.from_scene(scenes.make_scene(n, 5, -1.5, 1.5, mu, 0.4, 1, opacity_sd=3.0))
    cams, r = gs.Cameras(scenes.arc_cameras(large, 4.0, W, H)), raster()
    target = torch.rand(large, 3, H, W, generator=torch.Generator("cuda").manual_seed(4),
                        device="cuda")

    def both(c, t):
        out = r.forward(g, c, BG, own_buffers=True)
        loss = torch.zeros(1, dtype=torch.float64, device="cuda")
        grad = torch.empty_like(t)
        l1 = r.forward_l1(g, c, t, grad, loss, BG, keep_image=True, own_buffers=True)
        return out, l1, torch.sign(grad)

    whole, whole_l1, whole_sign = both(cams, target)
    mean, spread = shape(whole["lists"], cams, n)
    assert (mean < 40 and cams.n_segments() > 4_000) or (spread > 20 and
                                                         cams.n_segments() > 12_000)
    for v in range(0, large - 19, 40):
        part, part_l1, part_sign = both(cams.slice(v, 20), target[v:v + 20].contiguous())
        for k in ("image", "final_T", "n_contrib"):
            assert torch.equal(part[k], whole[k][v:v + 20]), k
            assert torch.equal(part_l1[k], whole_l1[k][v:v + 20]), k
        assert torch.equal(part_sign, whole_sign[v:v + 20])
