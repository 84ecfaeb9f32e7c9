"""Projection against the oracle over the view groups and the workgroup's
table of 16 views (partial, full, second), partial workgroups, and the
divisions that share a denominator at both ends of their range: covariances
up to the end of FP64, which cover every tile (the oracle's radius is an
int32, so it is not asked about those)."""
import numpy as np
import pytest

import oracle
from paper_2512_20943_amd import gs, scenes
from tests.gpu_helpers import projected_to_oracle, require_gpu, span_rows
from tests.test_gpu_parity import compare_projection

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 257, 1500])
@pytest.mark.parametrize("views", [1, 3, 16, 17, 34])
@pytest.mark.parametrize("tileset", ["rect", "tight", "spans"])
def test_projection_view_groups(n, views, tileset):
    require_gpu()
    print(f"project n={n} views={views} {tileset}", flush=True)
    scene = scenes.make_scene(n, n + views, -2.0, 2.0, -3.5, 0.7, 2)
    k = np.arange(n)
    for every, log_scale in ((5, 90.0), (7, 120.0), (11, 171.0)):
        scene["log_scale"][:, :n][:, k % every == every - 1] = log_scale
    scene["quat"][:, :n][:, k % 13 == 12] = 0.0
    scene["opacity"][:n][k % 17 == 16] = -9.0
    items = []
    for v in range(views):
        c = scenes.arc_cameras(1, 3.0 + 0.2 * v, 33 + 16 * (v % 3), 17 + 30 * (v % 4))
        items.append((c["R"][0], c["t"][0], c["f"][0], tuple(c["wh"][0])))
    cams = scenes.stack_cams(items)
    g, gc = gs.Gaussians.from_scene(scene), gs.Cameras(cams)
    proj = gs.Projected.empty(views, n, g.ld, "cuda")
    proj.options = {"rect": 0, "tight": gs.GS_PROJECT_TIGHT_RECT,
                    "spans": gs.GS_PROJECT_TIGHT_RECT | gs.GS_PROJECT_TILE_SPANS}[tileset]
    gs.gs_project(gs.default_context(), g, gc, proj)
    P_or, P_g = oracle.project(scene, cams, tileset), projected_to_oracle(proj)
    huge = scene["log_scale"][0, :n] > 80.0
    grid = (cams["wh"] + 15) // 16
    seen = 0
    for v in range(views):
        on = huge & (P_g["tiles"][v] > 0)
        seen += int(on.sum())
        assert (P_g["rect"][v, on] == np.array([0, 0, grid[v, 0], grid[v, 1]])).all()
        assert (P_g["tiles"][v, on] == grid[v].prod()).all()
    assert seen >= views * int((huge & (scene["opacity"][:n] > -5)).sum()) // 2

    def others(P):
        return {k: a[:, ~huge] if isinstance(a, np.ndarray) else a for k, a in P.items()}

    P_or, P_g = others(P_or), others(P_g)
    assert compare_projection(P_g, P_or) > 0
    (sp_g, rows_g), (sp_o, rows_o) = span_rows(P_g), span_rows(P_or)
    np.testing.assert_array_equal(sp_g, sp_o)
    np.testing.assert_array_equal(rows_g, rows_o)
