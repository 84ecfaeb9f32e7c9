"""Infinities and NaN in dL/dimage, and infinite colours: launches of every size
spread them to the same instances.  Large launches (one wave per tile) leave an
entry that no pixel of the tile composited at zero, so the small ones have to
as well."""
import numpy as np
import pytest
import torch

from paper_2512_20943_amd import gs, scenes
from paper_2512_20943_amd.raster import Rasterizer
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu

# 11 x 11 tiles a view: 4,840 tiles in all (one wave per tile), 121 and 242
# in launches of 1 and 2 (two waves per quadrant), 1,210 in launches of 10
# (one wave per quadrant)
W, H, VIEWS = 170, 165, 40
BG = (0.3, 0.1, 0.2)


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf"), "colours"])
@pytest.mark.parametrize("k", [1, 2, 10])
def test_only_composited_entries_become_nonfinite(value, k):
    require_gpu()
    print(f"non-finite dL/dimage {value} {k}", flush=True)
    scene = scenes.make_scene(3_000, 11, -2.0, 2.0, -3.0, 0.6, 1, opacity_sd=3.0)
    if value == "colours":
        scene["sh"][0, :, :3_000:300] = np.inf
    g = gs.Gaussians.from_scene(scene)
    cams = gs.Cameras(scenes.arc_cameras(VIEWS, 5.0, W, H))
    r = Rasterizer(ctx=gs.Context(torch.cuda.current_device()), capacity=1 << 22, tight_rect=True,
                   tile_spans=True)
    rng = np.random.default_rng(3)
    dimg = rng.uniform(-1, 1, (VIEWS, 3, H, W)).astype(np.float32)
    for v in range(VIEWS if value != "colours" else 0):
        for _ in range(12):
            dimg[v, rng.integers(3), rng.integers(H), rng.integers(W)] = value
    dimg = torch.from_numpy(dimg).cuda()

    def grads(c, d):
        out = r.forward(g, c, BG)
        grad = gs.Gaussians.zeros_like(g)
        ws = r.backward(g, c, out, d, grad, BG)
        return ws[: c.V * g.ld * 48].view(torch.float32).view(c.V, g.ld, 12)[:, :g.n, :9].clone()

    whole = grads(cams, dimg)
    bad = ~torch.isfinite(whole)
    assert 0 < int(bad.sum()) < bad.numel()
    for v in range(0, VIEWS, k):
        part = grads(cams.slice(v, k), dimg[v:v + k].contiguous())
        ref, ref_bad = whole[v:v + k], bad[v:v + k]
        part_bad = ~torch.isfinite(part)
        # an 8x4 half of a quadrant may skip an entry that the quadrant evaluates
        assert int((part_bad & ~ref_bad).sum()) == 0, f"view {v}"
        if k == 10:
            assert torch.equal(part_bad, ref_bad)
        # the finite rest as in the other tests of launch sizes
        a = torch.where(ref_bad | part_bad, 0.0, part).double()
        b = torch.where(ref_bad | part_bad, 0.0, ref).double()
        for q in range(9):
            assert (a[..., q] - b[..., q]).norm() <= 2.5e-5 * b[..., q].norm(), f"column {q}"
