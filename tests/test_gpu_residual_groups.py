"""The sent-update kernels take four texels at a time where planes and
buffers allow it: grids on both sides of that rule, ragged ends, and
misaligned buffers, bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_20943_amd import gs, scenes
from paper_2512_20943_amd.raster import frame_of
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu


def at_offset(a, off):
    """A device copy whose storage starts ``off`` elements into its buffer."""
    t = torch.from_numpy(np.ascontiguousarray(a))
    buf = torch.empty(t.numel() + off, dtype=t.dtype, device="cuda")
    out = buf[off:].view(t.shape)
    out.copy_(t)
    return out


# planes of 4 k texels (vector path; ragged at n) and not (one at a time), and
# planes whose buffers start off the alignment
@pytest.mark.parametrize("n,gw,gh,off", [
    (1, 2, 2, 0), (1_021, 32, 32, 0), (1_024, 32, 32, 0), (1_020, 33, 31, 0), (5, 7, 1, 0),
    (1_021, 32, 32, 1), (4_097, 68, 64, 0),
])
@pytest.mark.parametrize("bits", [8, 16])
def test_sent_update_bit_exact(n, gw, gh, off, bits):
    require_gpu()
    print(f"sent update n {n} grid {gw}x{gh} offset {off} bits {bits}", flush=True)
    ctx = gs.default_context()
    sc = scenes.make_scene(n, 2, -3, 3, -4, 0.5, 0)
    anchor = gs.Gaussians.from_scene(sc)
    frame = frame_of(anchor)
    P0 = np.zeros((8, gh, gw), np.float32)
    P0[3] = 1.0
    D = scenes.make_delta(n, gw, gh, 5)
    mask = scenes.prune_mask(D, n, 0.25)
    d_or, amax_or = oracle.residual_delta(D, P0, mask, n)
    q_or, s_or = oracle.quantize_delta(d_or, amax_or, bits)
    P_or = oracle.accumulate_sent(P0, oracle.dequantize_delta(q_or, s_or))
    f_or = oracle.apply(sc, P_or, np.ones((gh, gw), np.uint8), gw, gh)
    srv, cli = at_offset(P0, off), at_offset(P0, off)
    d = at_offset(np.full_like(P0, np.nan), off)
    q = at_offset(np.full(P0.shape, 99, np.int8 if bits == 8 else np.int16), off)
    amax, s = torch.zeros(8, device="cuda"), torch.empty(8, device="cuda")
    gs.gs_residual_delta(ctx, at_offset(D, off), srv, at_offset(mask, off), n, gw, gh, d, amax)
    gs.gs_quantize_delta(ctx, d, amax, bits, n, gw, gh, q, s, srv)
    gs.gs_apply_quantized_update(ctx, anchor, q, bits, s, cli, gw, gh, frame)
    q2 = torch.empty_like(q)
    gs.gs_quantize_delta(ctx, d, amax, bits, n, gw, gh, q2, s)  # without the running sum
    torch.cuda.synchronize()
    np.testing.assert_array_equal(d.cpu().numpy(), d_or)
    np.testing.assert_array_equal(amax.cpu().numpy(), amax_or)
    np.testing.assert_array_equal(q.cpu().numpy(), q_or)
    assert torch.equal(q, q2)
    np.testing.assert_array_equal(s.cpu().numpy(), s_or)
    for P in (srv, cli):
        np.testing.assert_array_equal(P.cpu().numpy().reshape(8, -1)[:, :n],
                                      P_or.reshape(8, -1)[:, :n])
        np.testing.assert_array_equal(P.cpu().numpy().reshape(8, -1)[:, n:],
                                      P0.reshape(8, -1)[:, n:])
    for k, t in (("mean", frame.mean), ("quat", frame.quat), ("opacity", frame.opacity)):
        np.testing.assert_array_equal(t.cpu().numpy()[..., :n], f_or[k][..., :n])


def test_a_nan_residual_shows_in_the_range():
    require_gpu()
    print("nan residual", flush=True)
    D, P = torch.zeros(8, 4, 4, device="cuda"), torch.zeros(8, 4, 4, device="cuda")
    D[2, 1, 1], D[4, 0, 0] = float("nan"), -3.0
    d, amax = torch.empty_like(D), torch.zeros(8, device="cuda")
    gs.gs_residual_delta(gs.default_context(), D, P,
                         torch.ones(4, 4, dtype=torch.uint8, device="cuda"), 16, 4, 4, d, amax)
    out = amax.cpu().numpy()
    assert np.isnan(out[2]) and out[4] == 3.0 and (out[[0, 1, 3, 5, 6, 7]] == 0).all()
