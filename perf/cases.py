"""The work a user of this framework has it do, as cases that can be timed.

Seven kinds, each through the calls that a program makes:

* ``step``: one training iteration -- projection, binning, compositing with
  the L1 term, backward, Adam -- written with the direct calls (``direct``),
  as torch autograd (``autograd``), or on the delta images of a frozen anchor
  with the temporal term (``delta``);
* ``view``: one delivered view: the frame's update applied, then rendered;
* ``burst``: requests that arrive together at the native view server;
* ``dssim``: the L1 + D-SSIM loss and its gradient;
* ``codec``: one sent update, at the server and at the client;
* ``compact``: low-opacity culling and the gather of the kept planes;
* ``sweep``: the pruning-level sweep of one frame.

Scenes have the repository's synthetic distributions (uniform means in a box,
normal log-scales, unit quaternions, normal opacity logits) and its camera
arcs; they are drawn on the GPU so that making them is quick.  ``exact`` is
an FP64 renderer of its own in plain torch.
"""
import math

import numpy as np
import torch

from paper_2512_20943_amd import gs, serve
from paper_2512_20943_amd.prune import PruningSweep
from paper_2512_20943_amd.raster import GSRenderL1, Rasterizer, frame_of

DEV = "cuda"
Y00 = 0.28209479177387814
# a late step of the schedule: the updates are small, so that the scene a
# pass sees stays the one that was drawn however many passes run
LR, STEP = 1e-6, 1000
TEMPORAL = 1e-3
CULL = 0.2173  # sigmoid of the normal's 10 % quantile: culls a tenth
RES = ((640, 480), (1280, 720), (1920, 1080))


def listed():
    return [
        # the smallest scene that is trained: latency and launches
        dict(name="step_small", kind="step", path="direct", n=10_000, deg=0, views=1, w=128,
             h=128, box=1.0, mu=-4.0, sd=0.5, radius=4.0),
        # a few views of odd size written with torch autograd, as a program
        # with a loss of its own around it would
        dict(name="step_autograd", kind="step", path="autograd", n=60_000, deg=2, views=3,
             w=641, h=483, box=3.0, mu=-4.0, sd=0.5, radius=5.0),
        # the per-frame training iteration: 20 views of 1352x1014
        dict(name="step_frame", kind="step", path="direct", n=300_000, deg=3, views=20, w=1352,
             h=1014, box=3.0, mu=-4.0, sd=0.5, radius=5.0),
        # the largest scene: cameras inside a cloud of 2 million
        dict(name="step_large", kind="step", path="direct", n=2_000_000, deg=3, views=8, w=1920,
             h=1080, box=6.0, mu=-4.5, sd=0.7, radius=5.0),
        # an in-group frame: the update trained on a frozen anchor
        dict(name="step_delta", kind="step", path="delta", n=120_000, deg=3, views=4, w=801,
             h=603, box=3.0, mu=-4.0, sd=0.5, radius=5.0),
        # one viewer's request, latency-bound
        dict(name="view_720p", kind="view", n=300_000, deg=3, w=1280, h=720, box=3.0, mu=-4.0,
             sd=0.5),
        # twelve requests of the three served sizes at once
        dict(name="serve_burst", kind="burst", n=300_000, deg=3, requests=12, frames=4, res=-1,
             box=3.0, mu=-4.0, sd=0.5),
        # Eq. (1) on the training step's 20 views
        dict(name="dssim_frame", kind="dssim", views=20, w=1352, h=1014),
        # and on a single view
        dict(name="dssim_view", kind="dssim", views=1, w=1352, h=1014),
        # a frame's update sent and received, 8-bit codes
        dict(name="codec_frame", kind="codec", n=300_000, bits=8),
        # keyframe compaction of all 59 planes
        dict(name="compact_frame", kind="compact", n=300_000, deg=3),
        # eleven pruning levels of a frame over four evaluation views
        dict(name="sweep_frame", kind="sweep", n=300_000, deg=3, views=4, w=1352, h=1014,
             levels=11, box=3.0, mu=-4.0, sd=0.5, radius=5.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "view", "burst", "dssim", "codec", "compact",
                       "sweep"])
    if kind == "step":
        w = _log(rng, 65, 1920)
        h = max(33, int(w * rng.uniform(0.5, 1.1)))
        n = _log(rng, 1_000, 1_000_000)
        most = max(1, min(20, int(16e6 / (w * h)), int(5e6 / n)))
        return dict(kind="step", path=rng.choice(["direct", "autograd", "delta"]), n=n,
                    deg=rng.randint(0, 3), views=rng.randint(1, most), w=w, h=h,
                    box=rng.choice([2.0, 3.0, 4.0]), mu=rng.choice([-4.5, -4.0]), sd=0.5,
                    radius=5.0)
    if kind == "view":
        w = _log(rng, 160, 3840)
        return dict(kind="view", n=_log(rng, 10_000, 2_000_000), deg=rng.randint(0, 3), w=w,
                    h=max(90, int(w * rng.uniform(0.5, 0.8))), box=rng.choice([3.0, 6.0]),
                    mu=-4.5, sd=rng.choice([0.5, 0.7]))
    if kind == "burst":
        return dict(kind="burst", n=_log(rng, 20_000, 300_000), deg=rng.randint(0, 3),
                    requests=rng.randint(1, 24), frames=rng.randint(1, 4),
                    res=rng.choice([-1, 0, 1, 2]), box=3.0, mu=-4.0, sd=0.5)
    if kind == "dssim":
        w = _log(rng, 65, 1920)
        h = max(33, int(w * rng.uniform(0.5, 1.1)))
        return dict(kind="dssim", views=rng.randint(1, max(1, min(20, int(24e6 / (w * h))))), w=w,
                    h=h)
    if kind == "codec":
        return dict(kind="codec", n=_log(rng, 5_000, 2_000_000), bits=rng.choice([8, 16]))
    if kind == "compact":
        return dict(kind="compact", n=_log(rng, 5_000, 2_000_000), deg=rng.randint(0, 3))
    w = _log(rng, 200, 1352)
    return dict(kind="sweep", n=_log(rng, 10_000, 300_000), deg=rng.randint(0, 3),
                views=rng.randint(1, 4), w=w, h=int(w * 0.75), levels=rng.randint(4, 11),
                box=3.0, mu=-4.0, sd=0.5, radius=5.0)


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _ld(n):
    return (n + 63) // 64 * 64


def _shapes(deg, ld):
    return ((3, ld), (3, ld), (4, ld), (ld,), ((deg + 1) ** 2, 3, ld))


def _planes(flat, deg, ld):
    out, o = [], 0
    for s in _shapes(deg, ld):
        out.append(flat[o:o + math.prod(s)].view(*s))
        o += math.prod(s)
    return out


def _scene(c, g):
    """All parameter planes in one buffer, as a trainer keeps them."""
    n, deg, ld = c["n"], c["deg"], _ld(c["n"])
    flat = torch.zeros(sum(math.prod(s) for s in _shapes(deg, ld)), device=DEV)
    mean, lsc, quat, opac, sh = _planes(flat, deg, ld)
    mean[:, :n] = (torch.rand(3, n, generator=g, device=DEV) * 2 - 1) * c.get("box", 3.0)
    lsc[:, :n] = torch.randn(3, n, generator=g, device=DEV) * c.get("sd", 0.5) + c.get("mu", -4.0)
    q = torch.randn(4, n, generator=g, device=DEV)
    quat[:, :n] = q / q.norm(dim=0, keepdim=True)
    quat[0, n:] = 1.0
    opac[:n] = torch.randn(n, generator=g, device=DEV)
    sh[0, :, :n] = (torch.rand(3, n, generator=g, device=DEV) - 0.5) / Y00
    if deg:
        sh[1:, :, :n] = 0.1 * torch.randn((deg + 1) ** 2 - 1, 3, n, generator=g, device=DEV)
    return flat


def _gaussians(c, flat):
    return gs.Gaussians(c["n"], c["deg"], _ld(c["n"]), *_planes(flat, c["deg"], _ld(c["n"])))


def _look(eye, w, h):
    """Camera at ``eye`` looking at the origin, 60-degree horizontal field."""
    eye = np.asarray(eye, np.float64)
    z = -eye / np.linalg.norm(eye)
    up = [0.0, 1.0, 0.0] if abs(z[1]) <= 0.99 else [0.0, 0.0, 1.0]
    x = np.cross(z, up)
    x /= np.linalg.norm(x)
    R = np.stack([x, np.cross(z, x), z])
    f = w / 2.0 / math.tan(math.radians(30.0))
    return R, -R @ eye, np.array([f, f, w / 2.0, h / 2.0]), (w, h)


def _arc(c, seed):
    """The views of a step: an even 120-degree arc, turned a little by the
    seed."""
    V, turn = c["views"], np.random.default_rng(seed).uniform(-0.1, 0.1)
    a = turn + (np.linspace(-math.pi / 3, math.pi / 3, V) if V > 1 else np.zeros(1))
    return [_look([c["radius"] * math.sin(t), 0.0, -c["radius"] * math.cos(t)], c["w"], c["h"])
            for t in a]


def _viewpoint(rng, w, h):
    d = rng.normal(size=3)
    return _look(rng.uniform(4.0, 6.0) * d / np.linalg.norm(d), w, h)


def _images(views, w, h, g, noise):
    """Image-like planes in [0, 1]: low-frequency cosines and noise."""
    x = torch.arange(w, device=DEV, dtype=torch.float32)
    y = torch.arange(h, device=DEV, dtype=torch.float32)[:, None]
    k = torch.rand(views, 3, 4, 3, 1, 1, generator=g, device=DEV)
    img = torch.full((views, 3, h, w), 0.4, device=DEV)
    for j in range(4):
        img += 0.15 * torch.cos(0.05 * k[:, :, j, 0] * x + 0.05 * k[:, :, j, 1] * y
                                + 6.28 * k[:, :, j, 2])
    return (img + noise * torch.randn(views, 3, h, w, generator=g, device=DEV)).clamp_(0, 1)


def _side(n):
    return int(math.ceil(math.sqrt(n)))


def _delta(n, g):
    """(8, gh, gw) delta images: identity update plus small motion."""
    s = _side(n)
    d = torch.zeros(8, s * s, device=DEV)
    d[3] = 1.0
    sd = torch.tensor([0.005] * 7 + [0.01], device=DEV)[:, None]
    d[:, :n] += sd * torch.randn(8, n, generator=g, device=DEV)
    return d.view(8, s, s)


def _mask(n, g, keep=0.7):
    s = _side(n)
    m = torch.zeros(s * s, dtype=torch.uint8, device=DEV)
    m[:n] = (torch.rand(n, generator=g, device=DEV) < keep).to(torch.uint8)
    return m.view(s, s)


def _raster(c):
    # capacity a program would start with; it grows on the first pass
    return Rasterizer(ctx=gs.Context(torch.cuda.current_device()), capacity=1 << 22,
                      tight_rect=True, tile_spans=True)


def _step_inputs(c, seed):
    g = _gen(seed)
    i = dict(flat=_scene(c, g), cams=_arc(c, seed),
             target=_images(c["views"], c["w"], c["h"], g, 0.1))
    if c["path"] == "delta":
        i["delta"], i["mask"] = _delta(c["n"], g), _mask(c["n"], g)
    return i


def prepare(case, seed):
    c = dict(case)
    kind = c["kind"]
    s = dict(c=c)
    if kind == "step":
        i = _step_inputs(c, seed)
        s.update(flat=i["flat"], cams=gs.Cameras.from_list(i["cams"]), target=i["target"],
                 raster=_raster(c), loss=torch.zeros(1, dtype=torch.float64, device=DEV))
        s["g"] = _gaussians(c, s["flat"])
        trained = s["flat"]
        if c["path"] == "delta":
            trained = s["delta"] = i["delta"]
            s["mask"], s["frame"] = i["mask"], frame_of(s["g"])
            s["grad"] = gs.Gaussians.zeros_like(s["g"])
        if c["path"] == "autograd":
            s["flat"].requires_grad_(True)
        else:
            s["dimg"] = torch.empty_like(s["target"])
            s["gflat"] = torch.zeros_like(trained)
            if c["path"] == "direct":
                s["grad"] = _gaussians(c, s["gflat"])
        s["m"], s["v"] = torch.zeros_like(trained.detach()), torch.zeros_like(trained.detach())
    elif kind == "view":
        g = _gen(seed)
        s["anchor"] = _gaussians(c, _scene(c, g))
        s["delta"], s["mask"] = _delta(c["n"], g), _mask(c["n"], g)
        s["frame"] = frame_of(s["anchor"])
        s["cams"] = gs.Cameras.from_list([_viewpoint(np.random.default_rng(seed), c["w"],
                                                     c["h"])])
        s["raster"] = _raster(c)
    elif kind == "burst":
        n, ld = c["n"], _ld(c["n"])
        host = [p.cpu().numpy() for p in _planes(_scene(c, _gen(seed)), c["deg"], ld)]
        scene = dict(zip(("mean", "log_scale", "quat", "opacity", "sh"), host), n=n,
                     deg=c["deg"], ld=ld)
        seq = serve.ResidentSequence(scene, c["frames"], seed=seed % 1000)
        rng = np.random.default_rng(seed)
        s["reqs"] = []
        for k in range(c["requests"]):
            w, h = RES[k % 3 if c["res"] < 0 else c["res"]]
            s["reqs"].append(serve.Request(k, int(rng.integers(c["frames"])),
                                           _viewpoint(rng, w, h), 0.0))
        s["server"] = serve.NativeServer(seq, 32 << 30)
    elif kind == "dssim":
        g = _gen(seed)
        s["target"] = _images(c["views"], c["w"], c["h"], g, 0.02)
        s["image"] = (s["target"] + 0.05 * torch.randn(s["target"].shape, generator=g,
                                                       device=DEV)).clamp_(0, 1)
        s["grad"] = torch.empty_like(s["image"])
        s["loss"] = torch.zeros(1, dtype=torch.float64, device=DEV)
        s["ws"] = torch.empty(gs.l1_dssim_workspace_size(3 * c["views"], c["h"], c["w"]),
                              dtype=torch.uint8, device=DEV)
        s["ctx"] = gs.Context(torch.cuda.current_device())
    elif kind == "codec":
        s.update(_codec_inputs(c, seed))
        s["anchor"] = _gaussians(dict(c, deg=0), s.pop("flat"))
        side = _side(c["n"])
        s["frame"], s["k"] = frame_of(s["anchor"]), 0
        s["cli"] = s["srv"].clone()
        s["d"] = torch.empty_like(s["srv"])
        s["amax"], s["scale"] = torch.zeros(8, device=DEV), torch.empty(8, device=DEV)
        s["q"] = torch.empty(8, side, side, device=DEV,
                             dtype=torch.int8 if c["bits"] == 8 else torch.int16)
        s["ctx"] = gs.Context(torch.cuda.current_device())
    elif kind == "compact":
        s["src"] = _scene(c, _gen(seed)).view(-1, _ld(c["n"]))
        s["idx"] = torch.zeros(c["n"], dtype=torch.int32, device=DEV)
        s["dst"] = torch.zeros_like(s["src"])
        s["ws"] = torch.empty(gs.cull_workspace_size(c["n"]), dtype=torch.uint8, device=DEV)
        s["ctx"] = gs.Context(torch.cuda.current_device())
    else:
        g = _gen(seed)
        anchor = _gaussians(c, _scene(c, g))
        s["ref"] = _images(c["views"], c["w"], c["h"], g, 0.05)
        s["sweep"] = PruningSweep(anchor, _delta(c["n"], g), _side(c["n"]), _side(c["n"]),
                                  gs.Cameras.from_list(_arc(c, seed)),
                                  ctx=gs.Context(torch.cuda.current_device()),
                                  levels=np.linspace(0.0, 1.0, c["levels"]))
    return s


def _codec_inputs(c, seed):
    """Accumulated deltas of eight successive frames, their masks, and what
    the client holds before the first of them (the identity update)."""
    g, n = _gen(seed), c["n"]
    side = _side(n)
    flat = _scene(dict(c, deg=0), g)
    D, walk = [], torch.zeros(8, side * side, device=DEV)
    walk[3] = 1.0
    ident = walk.clone().view(8, side, side)
    for _ in range(8):
        step = _delta(n, g).view(8, -1).clone()
        step[3] -= 1.0
        walk = walk + step
        D.append(walk.view(8, side, side))
    return dict(flat=flat, D=D, masks=[_mask(n, g) for _ in range(8)], srv=ident)


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(s):
    c = s["c"]
    kind = c["kind"]
    if kind == "step":
        return _run_step(s, c)
    if kind == "view":
        r = s["raster"]
        gs.gs_apply_frame_update(r.ctx, s["anchor"], s["delta"], s["mask"], _side(c["n"]),
                                 _side(c["n"]), s["frame"])
        out = r.forward(s["frame"], s["cams"])
        return dict(image=out["image"], final_T=out["final_T"], n_contrib=out["n_contrib"])
    if kind == "burst":
        s["server"].run(s["reqs"], keep_images=True)
        return [r.image for r in s["reqs"]]
    if kind == "dssim":
        s["loss"].zero_()
        gs.gs_l1_dssim_loss_grad(s["ctx"], s["image"], s["target"], s["grad"], s["loss"], s["ws"],
                                 0.2)
        return dict(loss=s["loss"], grad=s["grad"])
    if kind == "codec":
        n, side, x = c["n"], _side(c["n"]), s["ctx"]
        k = s["k"] % len(s["D"])
        s["k"] += 1
        s["amax"].zero_()
        gs.gs_residual_delta(x, s["D"][k], s["srv"], s["masks"][k], n, side, side, s["d"],
                             s["amax"])
        gs.gs_quantize_delta(x, s["d"], s["amax"], c["bits"], n, side, side, s["q"], s["scale"],
                             s["srv"])
        gs.gs_apply_quantized_update(x, s["anchor"], s["q"], c["bits"], s["scale"], s["cli"],
                                     side, side, s["frame"])
        f = s["frame"]
        return dict(d=s["d"], q=s["q"], scale=s["scale"], srv=s["srv"], cli=s["cli"],
                    mean=f.mean[:, :n], quat=f.quat[:, :n], opacity=f.opacity[:n])
    if kind == "compact":
        kept = gs.gs_cull_low_opacity(s["ctx"], s["src"][10], c["n"], CULL, s["idx"], s["ws"])
        gs.gs_gather_planes(s["ctx"], s["src"], s["idx"], kept, s["dst"])
        # the buffers hold zeros past the kept ones
        return dict(kept=kept, index=s["idx"], planes=s["dst"])
    out = s["sweep"].run(s["ref"])
    return dict(psnr=np.array(out["psnr"]), size=np.array(out["size"]),
                selected=out["selected"], usage=np.asarray(out["usage"]),
                masks=list(out["masks"]), images=out["images"])


def _run_step(s, c):
    r, cams, side = s["raster"], s["cams"], _side(c["n"])
    if c["path"] == "autograd":
        flat = s["flat"]
        flat.grad = None
        meta = (r, cams, c["n"], c["deg"], (0.0, 0.0, 0.0))
        loss = GSRenderL1.apply(*_planes(flat, c["deg"], _ld(c["n"])), s["target"], meta)
        loss.backward()
        p, grad = flat.detach(), flat.grad
        gs.gs_adam_step(r.ctx, p, grad, s["m"], s["v"], STEP, lr=LR)
        return dict(loss=loss.detach(), grad=grad, param=p, m=s["m"], v=s["v"])
    s["loss"].zero_()
    g = s["g"]
    if c["path"] == "delta":
        g = s["frame"]
        gs.gs_apply_frame_update(r.ctx, s["g"], s["delta"], s["mask"], side, side, g)
    out = r.forward_l1(g, cams, s["target"], s["dimg"], s["loss"])
    if c["path"] == "delta":
        r.backward(g, cams, out, s["dimg"], s["grad"], upd=(s["g"].quat, s["mask"], side, side),
                   dL_ddelta=s["gflat"], temporal=(TEMPORAL, s["delta"], s["loss"]))
        p = s["delta"]
    else:
        r.backward(g, cams, out, s["dimg"], s["grad"])
        p = s["flat"]
    gs.gs_adam_step(r.ctx, p, s["gflat"], s["m"], s["v"], STEP, lr=LR)
    return dict(loss=s["loss"], grad=s["gflat"], param=p, m=s["m"], v=s["v"],
                dimg=s["dimg"], final_T=out["final_T"], n_contrib=out["n_contrib"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _pairs(c, w, h, dist=5.0):
    """About how many (pixel, Gaussian) pairs one view composites: each
    Gaussian's visible footprint, at most some 72 a pixel (where the
    transmittance runs out)."""
    f = w / 2.0 / math.tan(math.radians(30.0))
    area = math.pi * 6.0 * ((f * math.exp(c["mu"]) / dist) ** 2 + 0.3)
    return min(72.0 * w * h, 0.6 * c["n"] * area)


def work(case):
    c = dict(case)
    kind = c["kind"]
    K = (c.get("deg", 0) + 1) ** 2
    per = 4.0 * (11 + 3 * K)  # bytes of one Gaussian's parameters
    if kind == "step":
        n, pix = c["n"], c["views"] * c["w"] * c["h"]
        pairs = c["views"] * _pairs(c, c["w"], c["h"], c["radius"])
        b = per * n + 12.0 * pix  # parameters and targets
        if c["path"] == "delta":
            b += 33.0 * n + 8 * 4.0 * n * 7  # update; gradient, Adam state
        else:
            b += per * n * 7  # gradient written, Adam's three planes read and written
        if c["path"] != "autograd":
            b += 20.0 * pix  # dL/dimage, final T, last contributor
        return dict(bytes=b, flops=pairs * (21 + 47) + 2000.0 * n * c["views"])
    if kind == "view":
        pix = c["w"] * c["h"]
        return dict(bytes=(per + 33.0) * c["n"] + 20.0 * pix,
                    flops=21 * _pairs(c, c["w"], c["h"]) + 1000.0 * c["n"])
    if kind == "burst":
        sizes = [RES[k % 3 if c["res"] < 0 else c["res"]] for k in range(c["requests"])]
        frames = min(c["frames"], c["requests"])
        return dict(bytes=(per + 33.0 * frames) * c["n"] + sum(12.0 * w * h for w, h in sizes),
                    flops=sum(21 * _pairs(c, w, h) + 1000.0 * c["n"] for w, h in sizes))
    if kind == "dssim":
        v = 3.0 * c["views"] * c["w"] * c["h"]
        return dict(bytes=12.0 * v, flops=v * (2 * 2 * 11 * 8 + 40))
    if kind == "codec":
        # D, D' read, mask; codes, d, both D' written; anchor read, frame written
        return dict(bytes=c["n"] * (32.0 * 7 + 1 + c["bits"]), flops=60.0 * c["n"])
    if kind == "compact":
        return dict(bytes=c["n"] * (per * 1.8 + 4.0 * 1.9), flops=float(c["n"]))
    pix = c["w"] * c["h"]
    lv = c["levels"] * c["views"]
    return dict(bytes=(per + 32.0) * c["n"] + 12.0 * pix * (c["views"] + lv),
                flops=(lv + c["views"]) * (21 * _pairs(c, c["w"], c["h"]) + 1000.0 * c["n"]))


# ---------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# ---------------------------------------------------------------------------

def _sh(deg, d):
    """Real orthonormal basis at unit directions d (n, 3), (n, K)."""
    x, y, z = d.unbind(1)
    Y = [torch.full_like(x, Y00)]
    if deg >= 1:
        a = math.sqrt(3 / (4 * math.pi))
        Y += [a * y, a * z, a * x]
    if deg >= 2:
        a, b, e = (math.sqrt(15 / (4 * math.pi)), math.sqrt(5 / (16 * math.pi)),
                   math.sqrt(15 / (16 * math.pi)))
        Y += [a * x * y, a * y * z, b * (3 * z * z - 1), a * x * z, e * (x * x - y * y)]
    if deg >= 3:
        a, b = math.sqrt(35 / (32 * math.pi)), math.sqrt(105 / (4 * math.pi))
        e, f = math.sqrt(21 / (32 * math.pi)), math.sqrt(7 / (16 * math.pi))
        Y += [a * y * (3 * x * x - y * y), b * x * y * z, e * y * (5 * z * z - 1),
              f * z * (5 * z * z - 3), e * x * (5 * z * z - 1), 0.5 * b * z * (x * x - y * y),
              a * x * (x * x - 3 * y * y)]
    return torch.stack(Y, 1)


def _project64(deg, mean, lsc, quat, opac, sh, cam):
    """Screen records (n, 9): px, py, A, B, C, opacity, r, g, b; depth, the
    tile rectangle (n, 4), visibility."""
    R, t, (fx, fy, cx, cy), (W, H) = cam
    R, t = (torch.tensor(np.asarray(a), dtype=torch.float64, device=DEV) for a in (R, t))
    w, x, y, z = (quat / quat.norm(dim=0)).unbind(0)
    Rq = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                      2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                      2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1)
    M = Rq.view(-1, 3, 3) * lsc.exp().t()[:, None, :]
    xc = mean.t() @ R.t() + t
    zc = xc[:, 2]
    ok = zc.detach() > 0.2
    zs = torch.where(ok, zc, torch.ones_like(zc))
    lx, ly = 1.3 * 0.5 * W / fx, 1.3 * 0.5 * H / fy
    # the clamped ratio enters the Jacobian; no gradient where it clamps
    u, v = (xc[:, 0] / zs).clamp(-lx, lx), (xc[:, 1] / zs).clamp(-ly, ly)
    o = torch.zeros_like(zs)
    J = torch.stack([fx / zs, o, -fx * u / zs, o, fy / zs, -fy * v / zs], 1).view(-1, 2, 3)
    T = J @ (R @ M)
    S = T @ T.transpose(1, 2)
    a, b, d = S[:, 0, 0] + 0.3, S[:, 0, 1], S[:, 1, 1] + 0.3
    det = a * d - b * b
    px, py = fx * xc[:, 0] / zs + cx, fy * xc[:, 1] / zs + cy
    dirs = mean.t() + (R.t() @ t)
    Y = _sh(deg, dirs / dirs.norm(dim=1, keepdim=True))
    rgb = (torch.einsum("nk,kcn->nc", Y, sh) + 0.5).clamp_min(0)
    rec = torch.cat([torch.stack([px, py, d / det, -b / det, a / det, torch.sigmoid(opac)], 1),
                     rgb], 1)
    with torch.no_grad():
        mid = 0.5 * (a + d)
        rad = (3 * (mid + (mid * mid - det).clamp_min(0.1).sqrt()).sqrt()).ceil()
        tx, ty = (W + 15) // 16, (H + 15) // 16
        rect = torch.stack([((px - rad) / 16).floor().clamp(0, tx),
                            ((py - rad) / 16).floor().clamp(0, ty),
                            (((px + rad) / 16).floor() + 1).clamp(0, tx),
                            (((py + rad) / 16).floor() + 1).clamp(0, ty)], 1).long()
        area = (rect[:, 2] - rect[:, 0]) * (rect[:, 3] - rect[:, 1])
        ok = ok & (det > 0) & (area > 0)
    return rec, zc.detach().float(), rect, ok


def _lists64(depth, rect, ok, W):
    """Instances in (tile, depth, id) order."""
    ids = ok.nonzero()[:, 0]
    r = rect[ids]
    w = r[:, 2] - r[:, 0]
    cnt = w * (r[:, 3] - r[:, 1])
    inst = torch.repeat_interleave(torch.arange(ids.numel(), device=DEV), cnt)
    local = torch.arange(inst.numel(), device=DEV) - (cnt.cumsum(0) - cnt)[inst]
    tile = (r[inst, 1] + local // w[inst]) * ((W + 15) // 16) + r[inst, 0] + local % w[inst]
    key = (tile << 32) | depth[ids].view(torch.int32).long()[inst]
    order = torch.sort(key, stable=True)[1]
    return ids[inst[order]], tile[order]


def _composite64(rec, gid, tile, W, H, pixel_fn):
    """Composites tile by tile; pixel_fn(px, py, colour (t, 256, 3), T) gets
    the pixels of a group of tiles."""
    tx, ty = (W + 15) // 16, (H + 15) // 16
    count = torch.bincount(tile, minlength=tx * ty)
    start = count.cumsum(0) - count
    order = torch.argsort(count)
    p = torch.arange(256, device=DEV)
    at, most = 0, count[order].tolist()
    while at < tx * ty:
        end = at + 1
        while end < tx * ty and (end + 1 - at) * max(1, most[end]) <= 40_000:
            end += 1
        tl, L = order[at:end], max(1, most[end - 1])
        at = end
        k = torch.arange(L, device=DEV)
        have = k[None] < count[tl][:, None]
        q = rec[gid[(start[tl][:, None] + k[None]).clamp(max=max(gid.numel() - 1, 0))]] \
            if gid.numel() else rec.new_zeros(tl.numel(), L, 9)
        x = ((tl % tx) * 16)[:, None] + (p % 16)[None]
        y = ((tl // tx) * 16)[:, None] + (p // 16)[None]
        dx = q[:, :, 0, None] - x[:, None, :]
        dy = q[:, :, 1, None] - y[:, None, :]
        power = -0.5 * (q[:, :, 2, None] * dx * dx + q[:, :, 4, None] * dy * dy) \
            - q[:, :, 3, None] * dx * dy
        raw = q[:, :, 5, None] * torch.exp(power.clamp(max=0))
        alpha = raw.clamp(max=0.99) * (have[:, :, None] & (raw.detach() >= 1 / 255)
                                       & (power.detach() <= 0))
        T = torch.exp(torch.cumsum(torch.log1p(-alpha), 1))
        a = alpha * (T.detach() >= 1e-4)
        T = torch.exp(torch.cumsum(torch.log1p(-a), 1))
        before = torch.cat([torch.ones_like(T[:, :1]), T[:, :-1]], 1)
        pixel_fn(x, y, torch.einsum("tlp,tlc->tpc", a * before, q[:, :, 6:9]), T[:, -1])


def _frame64(c, flat, delta, mask):
    """The frame an update makes of an anchor, rounded once to 32 bits."""
    n = c["n"]
    mean, lsc, quat, opac, sh = (p[..., :n].double() for p in _planes(flat, c["deg"],
                                                                        _ld(n)))
    if delta is not None:
        d, k = delta.reshape(8, -1)[:, :n].double(), mask.view(-1)[:n].bool()
        if d.requires_grad:
            d.retain_grad()
        w, x, y, z = d[3], d[4], d[5], d[6]
        W, X, Y, Z = quat
        moved = torch.stack([w * W - x * X - y * Y - z * Z, w * X + x * W + y * Z - z * Y,
                             w * Y - x * Z + y * W + z * X, w * Z + x * Y - y * X + z * W])
        once = lambda v: v + (v.detach().float().double() - v.detach())  # noqa: E731
        mean = torch.where(k, once(mean + d[:3]), mean)
        quat = torch.where(k, once(moved), quat)
        opac = torch.where(k, once(opac + d[7]), opac)
    return mean, lsc, quat, opac, sh


def _render64(c, planes, cam):
    W, H = cam[3]
    with torch.no_grad():
        rec, depth, rect, ok = _project64(c["deg"], *planes, cam)
        gid, tile = _lists64(depth, rect, ok, W)
        img, fT = (torch.zeros(s, H, W, dtype=torch.float64, device=DEV) for s in (3, 1))

        def put(x, y, col, T):
            m = (x < W) & (y < H)
            img[:, y[m], x[m]] = col[m].t()
            fT[0, y[m], x[m]] = T[m]

        _composite64(rec, gid, tile, W, H, put)
    return img, fT[0]


def _adam64(p, g):
    m, v = 0.1 * g, 0.001 * g * g
    up = (m / (1 - 0.9 ** STEP)) / ((v / (1 - 0.999 ** STEP)).sqrt() + 1e-8)
    return dict(grad=g, param=p.double() - LR * up, m=m, v=v)


def _exact_step(c, seed):
    i, n, ld = _step_inputs(c, seed), c["n"], _ld(c["n"])
    delta = i.get("delta")
    lead = (delta if delta is not None else i["flat"]).double().requires_grad_(True)
    V, W, H = c["views"], c["w"], c["h"]
    dimg = torch.zeros(V, 3, H, W, dtype=torch.float64, device=DEV)
    fT = torch.zeros(V, H, W, dtype=torch.float64, device=DEV)
    loss, count = 0.0, V * 3 * H * W
    for v, cam in enumerate(i["cams"]):
        planes = _frame64(c, i["flat"], lead, i["mask"]) if delta is not None \
            else _frame64(c, lead, None, None)
        rec, depth, rect, ok = _project64(c["deg"], *planes, cam)
        gid, tile = _lists64(depth, rect, ok, W)
        leaf = rec.detach().requires_grad_(True)

        def pixels(x, y, col, T):
            nonlocal loss
            m = (x < W) & (y < H)
            d = col[m] - i["target"][v][:, y[m], x[m]].t().double()
            part = d.abs().sum() / count
            if part.requires_grad:
                part.backward()
            loss += float(part)
            dimg[v][:, y[m], x[m]] = d.detach().sign().t() / count
            fT[v, y[m], x[m]] = T[m].detach()

        _composite64(leaf, gid, tile, W, H, pixels)
        if leaf.grad is not None:
            rec.backward(torch.where(ok[:, None], leaf.grad, torch.zeros_like(leaf.grad)))
    grad = torch.zeros_like(lead) if lead.grad is None else torch.nan_to_num(lead.grad)
    if delta is not None:
        e = torch.zeros_like(grad.view(8, -1))
        e[3] = 1.0
        r = (lead.detach().view(8, -1) - e)[:, :n]
        grad.view(8, -1)[:, :n] += TEMPORAL * r.sign()
        loss += TEMPORAL * float(r.abs().sum())
    out = dict(loss=torch.tensor([loss], dtype=torch.float64),
               **_adam64(lead.detach(), grad))
    if c["path"] == "autograd":
        out["loss"] = out["loss"][0]
        return out
    return dict(out, dimg=dimg, final_T=fT, n_contrib=None)


def _windowed(x, wts):
    """11 x 11 separable window with zero padding over (H, W)."""
    p = torch.nn.functional.pad(x, (5, 5, 5, 5))
    p = sum(wts[k] * p[:, k:k + x.shape[1]] for k in range(11))
    return sum(wts[k] * p[k:k + x.shape[0]] for k in range(11))


def _exact_dssim(c, seed):
    s = prepare(c, seed)
    wts = np.exp(-np.arange(-5, 6) ** 2 / (2 * 1.5 ** 2))
    wts = (wts / wts.sum()).tolist()
    H, W = c["h"], c["w"]
    img, tgt = s["image"].view(-1, H, W), s["target"].view(-1, H, W)
    grad = torch.empty(img.shape, dtype=torch.float64, device=DEV)
    loss, count = 0.0, img.numel()
    for k in range(img.shape[0]):
        x, y = img[k].double().requires_grad_(True), tgt[k].double()
        mx, my = _windowed(x, wts), _windowed(y, wts)
        sx, sy = _windowed(x * x, wts) - mx * mx, _windowed(y * y, wts) - my * my
        sxy = _windowed(x * y, wts) - mx * my
        S = (2 * mx * my + 1e-4) * (2 * sxy + 9e-4) / ((mx * mx + my * my + 1e-4)
                                                      * (sx + sy + 9e-4))
        part = (0.8 * (x - y).abs().sum() + 0.2 * (1 - S).sum()) / count
        part.backward()
        loss += float(part)
        grad[k] = x.grad
    return dict(loss=torch.tensor([loss], dtype=torch.float64), grad=grad.view(s["image"].shape))


def _exact_codec(c, seed):
    s = _codec_inputs(c, seed)
    n, top = c["n"], 2 ** (c["bits"] - 1) - 1
    keep = torch.zeros_like(s["masks"][0].view(-1), dtype=torch.float64)
    keep[:n] = s["masks"][0].view(-1)[:n].double()
    old = s["srv"].view(8, -1).double()
    d = (s["D"][0].view(8, -1).double() - old) * keep
    scale = d.abs().amax(1) / top
    code = (d / scale[:, None]).round().clamp(-top, top)
    new = old.clone()
    new[:, :n] += (code * scale[:, None])[:, :n]
    flat = dict(c, deg=0)
    mean, _, quat, opac, _ = _frame64(flat, s["flat"], new, torch.ones_like(s["masks"][0]))
    shape = s["srv"].shape
    return dict(d=d.view(shape), q=None, scale=scale, srv=new.view(shape), cli=new.view(shape),
                mean=mean, quat=quat, opacity=opac)


def exact(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind == "step":
        # about the pairs that 20 seconds allow
        if c["views"] * c["w"] * c["h"] > 2.5e6 or c["views"] * c["n"] > 1e6:
            return None
        return _exact_step(c, seed)
    if kind == "view":
        if c["n"] > 500_000 or c["w"] * c["h"] > 1.5e6:
            return None
        s = prepare(c, seed)
        flat = torch.cat([p.reshape(-1) for p in s["anchor"].planes()])
        cam = _viewpoint(np.random.default_rng(seed), c["w"], c["h"])
        img, fT = _render64(c, _frame64(c, flat, s["delta"], s["mask"]), cam)
        return dict(image=img[None], final_T=fT[None], n_contrib=None)
    if kind == "dssim":
        return _exact_dssim(c, seed)
    if kind == "codec":
        return _exact_codec(c, seed)
    if kind == "compact":
        src = _scene(c, _gen(seed)).view(-1, _ld(c["n"]))
        # decided on the logit in 64 bits, as sigmoid(logit) >= CULL
        thr = np.float64(np.float32(CULL))
        keep = src[10, :c["n"]].double() >= math.log(thr / (1.0 - thr))
        dst = torch.zeros_like(src, dtype=torch.float64)
        dst[:, :int(keep.sum())] = src[:, :c["n"]][:, keep].double()
        return dict(kept=None, index=None, planes=dst)
    return None
