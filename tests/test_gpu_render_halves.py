"""The compositing kernels of small launches (two waves per quadrant) against
those of large ones: views of partial tiles, one launch of many against
launches of few."""
import numpy as np
import pytest
import torch

from paper_2512_20943_amd import gs, scenes
from paper_2512_20943_amd.raster import Rasterizer
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu

# 11 x 11 tiles a view, the last row and column partial: 4,840 tiles in all,
# 121 and 242 in the small launches
W, H, VIEWS = 170, 165, 40
BG = (0.3, 0.1, 0.2)


@pytest.fixture(scope="module", params=["opaque", "thin"])
def views(request):
    require_gpu()
    if request.param == "opaque":  # opacities at the cap, pixels that stop early
        scene = scenes.make_scene(6_000, 11, -2.0, 2.0, -2.6, 0.6, 1, opacity_sd=5.0)
    else:
        scene = scenes.make_scene(3_000, 12, -2.0, 2.0, -3.2, 0.6, 1)
        scene["opacity"][:3_000] -= 2.0
    g = gs.Gaussians.from_scene(scene)
    cams = gs.Cameras(scenes.arc_cameras(VIEWS, 5.0, W, H))
    r = Rasterizer(ctx=gs.Context(torch.cuda.current_device()), capacity=1 << 22, tight_rect=True,
                   tile_spans=True)
    return request.param, r, g, cams


@pytest.mark.parametrize("k", [1, 2])
def test_forward_bits(views, k):
    name, r, g, cams = views
    print(f"halves forward {name} {k}", flush=True)
    whole = r.forward(g, cams, BG, own_buffers=True)
    target = torch.rand(VIEWS, 3, H, W, generator=torch.Generator("cuda").manual_seed(3),
                        device="cuda")
    for v in range(0, VIEWS, 8):
        c = cams.slice(v, k)
        part = r.forward(g, c, BG)
        for key in ("image", "final_T", "n_contrib"):
            assert torch.equal(whole[key][v:v + k], part[key]), key
        grad, loss = torch.empty_like(target[v:v + k]), torch.zeros(1, dtype=torch.float64,
                                                                    device="cuda")
        t = target[v:v + k].contiguous()
        part = r.forward_l1(g, c, t, grad, loss, keep_image=True)
        plain = r.forward(g, c, own_buffers=True)  # forward_l1's background is 0
        for key in ("image", "final_T", "n_contrib"):
            assert torch.equal(plain[key], part[key]), key
        d = plain["image"] - t
        assert torch.equal(torch.sign(grad), torch.sign(d))
        # FP64 sum of the same FP32 differences
        assert abs(float(loss) - float(d.abs().double().mean())) <= 1e-12


@pytest.mark.parametrize("k", [1, 2])
def test_backward_agrees(views, k):
    """Screen-space gradients of 40 views in one launch (one wave per tile) and
    in launches of k.  Both evaluate the same pairs; a term's products are
    rounded in another order (4 ulp) and at most 256 of them are added in
    another tree (10 ulp), on sums whose cancellation averages below 30 in
    norm: 14 * 30 * 2^-24 = 2.5e-5."""
    name, r, g, cams = views
    n = g.n
    dimg = torch.from_numpy(np.random.default_rng(9).uniform(-1, 1, (VIEWS, 3, H, W))
                            .astype(np.float32)).cuda()
    print(f"halves backward {name} {k}", flush=True)

    def grads(c, d):
        out = r.forward(g, c, BG)
        grad = gs.Gaussians.zeros_like(g)
        ws = r.backward(g, c, out, d, grad, BG)
        return ws[: c.V * g.ld * 48].view(torch.float32).view(c.V, g.ld, 12)[:, :n, :9].clone()

    whole = grads(cams, dimg).double()
    for v in range(0, VIEWS, 8):
        part = grads(cams.slice(v, k), dimg[v:v + k].contiguous()).double()
        for q in range(9):
            a, b = part[:, :, q], whole[v:v + k, :, q]
            assert (a - b).norm() <= 2.5e-5 * b.norm(), f"column {q} of view {v}"


@pytest.mark.parametrize("k", [1, 9, 20, 40])
def test_l1_sum_over_tiles(views, k):
    """The loss of 121 k tiles (1,089: a second step of the one workgroup that
    adds the partials, 4,840: its unrolled steps)."""
    name, r, g, cams = views
    print(f"l1 sum {name} {k}", flush=True)
    c = cams.slice(0, k)
    target = torch.rand(k, 3, H, W, generator=torch.Generator("cuda").manual_seed(k), device="cuda")
    loss = torch.full((1,), 0.5, dtype=torch.float64, device="cuda")
    out = r.forward_l1(g, c, target, torch.empty_like(target), loss, keep_image=True)
    want = 0.5 + float((out["image"] - target).abs().double().mean())
    # FP64 sums of the same FP32 differences
    assert abs(float(loss) - want) <= 1e-12


@pytest.mark.parametrize("w,h", [(1920, 1080), (640, 480)])
def test_backward_with_and_without_an_order_of_tiles(w, h):
    """48 splats in 8,160 and 1,200 tiles: the gradient records of 64 columns
    are too small for the tiles' order, those of 4,096 (the rest behind the
    camera) hold it.  The same rows either way, so the same bits."""
    require_gpu()
    print(f"order {w}x{h}", flush=True)
    scene = scenes.make_scene(48, 2, -1.0, 1.0, -1.5, 0.6, 1)
    more = scenes.make_scene(4_000, 3, -1.0, 1.0, -4.0, 0.5, 1)
    more["mean"][2, :4_000] = -50.0
    for k in ("mean", "log_scale", "quat", "opacity", "sh"):
        more[k][..., :48] = scene[k][..., :48]
    cams = gs.Cameras(scenes.axis_camera(w, h, 4.0))
    dimg = torch.rand(1, 3, h, w, generator=torch.Generator("cuda").manual_seed(1), device="cuda")

    def grads(sc):
        g = gs.Gaussians.from_scene(sc)
        r = Rasterizer(ctx=gs.Context(torch.cuda.current_device()), capacity=1 << 20)
        out = r.forward(g, cams, BG)
        grad = gs.Gaussians.zeros_like(g)
        r.backward(g, cams, out, dimg, grad, BG)
        return [p[..., :48].clone() for p in grad.planes()]

    for a, b in zip(grads(scene), grads(more)):
        assert a.abs().max() > 0 and torch.equal(a, b)
