"""The compositing kernels on both sides of the rules that choose between
them by the number of tiles of a launch: one launch over many small ragged
views (above the limits) against the same views in smaller launches (below
them), through the C ABI."""
import numpy as np
import pytest
import torch

from paper_2512_20943_amd import gs, scenes
from paper_2512_20943_amd.raster import Rasterizer
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu

# 11 x 11 tiles a view, the last row and column partial: 67,760 tiles in all,
# above both forward limits, and 16,940 a part, below them
W, H, VIEWS, PARTS = 170, 165, 560, 4


@pytest.fixture(scope="module")
def many_views():
    require_gpu()
    scene = scenes.make_scene(3_000, 11, -2.0, 2.0, -3.0, 0.6, 1, opacity_sd=3.0)
    g = gs.Gaussians.from_scene(scene)
    cams = gs.Cameras(scenes.arc_cameras(VIEWS, 5.0, W, H))
    ctx = gs.Context(torch.cuda.current_device())
    r = Rasterizer(ctx=ctx, capacity=1 << 22, tight_rect=True, tile_spans=True)
    rng = np.random.default_rng(5)
    target = torch.from_numpy(rng.uniform(0, 1, (VIEWS, 3, H, W)).astype(np.float32)).cuda()
    return r, g, cams, target


def parts(cams):
    k = VIEWS // PARTS
    return [(slice(i * k, (i + 1) * k), cams.slice(i * k, k)) for i in range(PARTS)]


def test_forward_is_the_same_in_large_and_small_launches(many_views):
    r, g, cams, _ = many_views
    print(f"forward split: {VIEWS} views {W}x{H}", flush=True)
    bg = (0.1, 0.2, 0.3)
    whole = r.forward(g, cams, bg, own_buffers=True)
    assert cams.n_segments() > 66_000
    for sl, c in parts(cams):
        part = r.forward(g, c, bg)
        for k in ("image", "final_T", "n_contrib"):
            assert torch.equal(whole[k][sl], part[k]), k


def test_fused_l1_forward_is_the_same_in_large_and_small_launches(many_views):
    r, g, cams, target = many_views
    print(f"fused L1 split: {VIEWS} views {W}x{H}", flush=True)
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    grad = torch.empty_like(target)
    whole = r.forward_l1(g, cams, target, grad, loss, keep_image=True, own_buffers=True)
    mean = 0.0
    for sl, c in parts(cams):
        lp = torch.zeros_like(loss)
        gp = torch.empty_like(target[sl])
        part = r.forward_l1(g, c, target[sl], gp, lp, keep_image=True)
        for k in ("image", "final_T", "n_contrib"):
            assert torch.equal(whole[k][sl], part[k]), k
        assert torch.equal(torch.sign(grad[sl]), torch.sign(gp))
        mean += float(lp) / PARTS
    # the same FP64 partial sums, added in another order
    assert abs(float(loss) - mean) <= 1e-13 * mean


def test_batched_launch_is_the_same_above_and_below_its_limit(many_views):
    r, g, cams, _ = many_views
    print(f"batched split: {VIEWS} views {W}x{H}", flush=True)
    ctx = r.ctx
    ref = r.forward(g, cams, own_buffers=True)["image"]

    def batched(c):
        proj = r.project(g, c)
        lists = r.bin_sort(proj, c)
        out = torch.full((c.V, 3, H, W), -7.0, device="cuda")
        ws = torch.empty(gs.render_batched_workspace_size(c.V), dtype=torch.uint8, device="cuda")
        gs.gs_render_fwd_batched(ctx, proj, lists, c, (0.0, 0.0, 0.0), out, ws)
        return out

    assert torch.equal(batched(cams), ref)
    for sl, c in parts(cams):
        assert torch.equal(batched(c), ref[sl])


def test_backward_agrees_in_large_and_small_launches(many_views):
    """Screen-space gradients per (view, Gaussian) of 40 views in one launch
    (4,840 tiles, one wave per tile) and in parts of 10 (1,210 tiles, one
    wave per quadrant).  Both evaluate the same pairs; a term's products are
    rounded in another order (4 ulp) and at most 256 of them are added in
    another tree (10 ulp), on sums whose cancellation averages below 30 in
    norm: 14 * 30 * 2^-24 = 2.5e-5."""
    r, g, cams, _ = many_views
    n, V, k = g.n, 40, 10
    c40 = cams.slice(100, V)
    rng = np.random.default_rng(9)
    dimg = torch.from_numpy(rng.uniform(-1, 1, (V, 3, H, W)).astype(np.float32)).cuda()
    bg = (0.3, 0.1, 0.2)

    def grads(c, d):
        out = r.forward(g, c, bg)
        grad = gs.Gaussians.zeros_like(g)
        ws = r.backward(g, c, out, d, grad, bg)
        g2 = ws[: c.V * g.ld * 48].view(torch.float32).view(c.V, g.ld, 12)[:, :n, :9]
        return g2.clone().double(), [p.double() for p in grad.planes()]

    print(f"backward split: {V} views {W}x{H}", flush=True)
    whole, total = grads(c40, dimg)
    summed = [torch.zeros_like(p) for p in total]
    for v in range(0, V, k):
        part, planes = grads(c40.slice(v, k), dimg[v:v + k].contiguous())
        for q in range(9):
            a, b = part[:, :, q], whole[v:v + k, :, q]
            assert (a - b).norm() <= 2.5e-5 * b.norm(), f"column {q} of views {v}"
        for s, p in zip(summed, planes):
            s += p
    for s, p in zip(summed, total):
        assert (s - p).norm() <= 5e-5 * p.norm()
