"""Where the native server writes its images: in place into any part of a
device buffer, left out for a request without one, and by copies in the
batch's order (by frame) where images of one batch overlap."""
import ctypes

import pytest
import torch

from paper_2512_20943_amd import gs, scenes, serve
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu

WH = ((64, 48), (31, 17), (200, 150))


@pytest.fixture(scope="module")
def seq():
    require_gpu()
    return serve.ResidentSequence(scenes.make_scene(5_000, 11, -3.0, 3.0, -4.0, 0.5, 1), 6, seed=3)


def offsets(sizes, layout):
    """Float offset of every image into one buffer, or None."""
    packed = [sum(sizes[:k]) for k in range(len(sizes))]
    if layout == "odd":           # 4-byte aligned only
        return [o + 2 * k + 1 for k, o in enumerate(packed)]
    if layout == "missing":
        return [None if k % 3 == 1 else o for k, o in enumerate(packed)]
    if layout == "shared":        # two requests with the same image pointer
        return [packed[1] if k == 2 else o for k, o in enumerate(packed)]
    if layout == "overlapping":   # neighbours share their last and first values
        return [o - 7 * k for k, o in enumerate(packed)]
    return packed


@pytest.mark.parametrize("plain", [False, True])
@pytest.mark.parametrize("layout", ["packed", "odd", "missing", "shared", "overlapping"])
def test_image_targets(seq, layout, plain):
    print(f"targets {layout} plain={plain}", flush=True)
    # one worker and frames in request order: images land in request order
    reqs = serve.make_trace(6, 1e6, None, 4, seq.n_frames, 21, resolutions=WH)
    for k, r in enumerate(reqs):
        r.frame = k
    alone = serve.PlainRenderer(seq)
    sizes = [3 * r.wh[0] * r.wh[1] for r in reqs]
    at = offsets(sizes, layout)
    buf = torch.full((sum(sizes) + 64,), -1.0, device="cuda")
    want = buf.clone()
    for r, o, s in zip(reqs, at, sizes):
        if o is not None:
            want[o:o + s] = alone.render(r).reshape(-1)
    srv = serve.NativeServer(seq, budget_bytes=8 << 30, max_batch=16, n_workers=1,
                             inline_singletons=False)
    n = len(reqs)
    c = (gs.GsRequest * n)()
    for k, r in enumerate(reqs):
        srv._camera(r.cam, c[k].cam)
        c[k].frame, c[k].arrival_s = r.frame, 0.0
    ptrs = (ctypes.c_void_p * n)(*[None if o is None else buf.data_ptr() + 4 * o for o in at])
    ts, td = (ctypes.c_double * n)(), (ctypes.c_double * n)()
    torch.cuda.synchronize()
    assert srv.lib.gs_server_run(srv.handle, c, n, int(plain), ts, td, ptrs) == gs.GS_OK
    assert torch.equal(buf, want)
    srv.close()
