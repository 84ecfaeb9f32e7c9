"""The projection's table of 16 views' constants past its first slot: groups of
16, 17, 33 and 40 views, which take enough Gaussians that the launch is not
split into more groups.  A view projected alone uses slot 0 only, and gives the
same bits; a part of each view is compared with the oracle as well.  Then the
lower end of the shared divisions."""
import re
from pathlib import Path

import numpy as np
import pytest
import torch

import oracle
from paper_2512_20943_amd import gs, scenes
from tests.gpu_helpers import projected_to_oracle, require_gpu, span_rows
from tests.test_gpu_parity import compare_projection

pytestmark = pytest.mark.gpu

SOURCE = Path(gs.__file__).parent / "csrc" / "gs_project.hip"


def views_per_group(n, views):
    """launch_project's rule, with the number of waves it aims at from there."""
    aim = int(re.search(r"\((\d+) \+ waves - 1\) / waves", SOURCE.read_text()).group(1))
    waves = 4 * -(-n // 256)
    groups = min(views, max(1, -(-aim // waves)))
    return -(-views // groups)


def cameras(views):
    items = []
    for v in range(views):
        c = scenes.arc_cameras(1, 3.0 + 0.1 * v, 33 + 16 * (v % 3), 17 + 30 * (v % 4),
                               azimuth_deg=90.0)
        items.append((c["R"][0], c["t"][0] + 0.01 * v, c["f"][0] * (1.0 + 0.02 * v),
                      tuple(c["wh"][0])))
    return scenes.stack_cams(items)


@pytest.mark.parametrize("n,views,per", [
    (262_145, 16, 16), (262_145, 17, 17), (262_145, 33, 33), (262_145, 40, 40),
    (131_073, 40, 20)])  # two groups, the second from the middle of the views on
def test_tables_past_their_first_slot(n, views, per):
    require_gpu()
    print(f"project table n={n} views={views}", flush=True)
    assert views_per_group(n, views) == per
    scene = scenes.make_scene(n, views, -2.0, 2.0, -3.5, 0.7, 1)
    cams = cameras(views)
    g, gc = gs.Gaussians.from_scene(scene), gs.Cameras(cams)
    ctx = gs.default_context()

    def project(c):
        out = gs.Projected.empty(c.V, n, g.ld, "cuda")
        out.options = gs.GS_PROJECT_TIGHT_RECT | gs.GS_PROJECT_TILE_SPANS
        gs.gs_project(ctx, g, c, out)
        return out

    whole = project(gc)
    for v in range(views):
        alone = project(gc.slice(v, 1))
        for k in ("splat", "rect", "tiles_touched", "depth_bits", "flags"):
            a, b = getattr(whole, k)[v, :n], getattr(alone, k)[0, :n]
            if a.dtype == torch.float32:
                a, b = a.view(torch.int32), b.view(torch.int32)
            assert torch.equal(a, b), f"{k} of view {v}"
    few = 300
    part = scenes.subset(scene, few)
    P_g = projected_to_oracle(whole)
    P_g = {k: (a[:, :few] if isinstance(a, np.ndarray) else a) for k, a in P_g.items()}
    assert compare_projection({**P_g, "n": few}, oracle.project(part, cams, "spans")) > 0


@pytest.mark.parametrize("tileset", ["rect", "tight", "spans"])
@pytest.mark.parametrize("isotropic", [False, True])
def test_gaussians_on_the_cameras_axes(tileset, isotropic):
    """Zeros of both signs and numerators at the lower end of the range in the
    quotients that share a denominator."""
    require_gpu()
    print(f"on the axes, {tileset}, isotropic {isotropic}", flush=True)
    n = 2_000
    scene = scenes.make_scene(n, 3, -1.0, 1.0, -3.0, 0.5, 1)
    tiny = np.array([0.0, -0.0, 1e-30, -1e-38, 1e-44], np.float32)
    scene["mean"][0, :n:2] = tiny[np.arange(n // 2) % 5]
    scene["mean"][1, :n:3] = tiny[np.arange(-(-n // 3)) % 4]
    if isotropic:
        scene["quat"][:, :n] = np.array([[1.0], [0.0], [0.0], [0.0]])
        scene["log_scale"][:, :n] = scene["log_scale"][0, :n]
    cams = scenes.axis_camera(200, 150, 4.0)
    cams["t"][0, 0] = -0.0
    g, gc = gs.Gaussians.from_scene(scene), gs.Cameras(cams)
    proj = gs.Projected.empty(1, n, g.ld, "cuda")
    proj.options = {"rect": 0, "tight": gs.GS_PROJECT_TIGHT_RECT,
                    "spans": gs.GS_PROJECT_TIGHT_RECT | gs.GS_PROJECT_TILE_SPANS}[tileset]
    gs.gs_project(gs.default_context(), g, gc, proj)
    P_g, P_or = projected_to_oracle(proj), oracle.project(scene, cams, tileset)
    assert compare_projection(P_g, P_or) > n // 2
    for a, b in zip(span_rows(P_g), span_rows(P_or)):
        np.testing.assert_array_equal(a, b)
