"""What the framework's speed is measured on: passes through its public entry
points (raster.forward / backward / render, step.TrainStep, deform.DeformNet)
over the range of scenes, images and options that its users render and train.

The scenes are synthetic, in the regime of indoor time-of-flight captures
(30 MHz, about 5 m unambiguous range): Gaussians uniform in the camera's view
at 0.5 to 4.5 m, standard deviations of a few centimetres, opacities
sigmoid(N(0, 1)), velocities of decimetres per second.  Upstream gradients are
N(0, 1) on every rendered element.

    listed()            the cases that are reported
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs, workspaces and weights, on the GPU
    run(state)          one pass, and its outputs
    work(case)          bytes and FLOP the pass cannot do without
    exact(case, seed)   the outputs in 64 bits by plain torch, where small enough
"""
import ctypes
import math

import torch

from paper_2505_05356_amd import deform, raster, step
from paper_2505_05356_amd._lib import FIELDS

LIGHT = 299_792_458.0
PHASES = (0.0, 0.5 * math.pi, math.pi, 1.5 * math.pi)
FREQS = (30e6, 60e6, 20e6, 50e6)
_STREAMS = {}


# ----------------------------------------------------------------------------
# Cases
# ----------------------------------------------------------------------------

def _scene(kind, n, frames, width, height, **more):
    """A rendering case: kind is "view" (forward only), "fwdbwd" (forward and
    backward on kept buffers), "render" (the autograd entry point, which
    allocates its outputs and checks the pair count) or "train" / "trainnet"
    (one optimisation step, captured once and replayed).  size: the median
    standard deviation of a Gaussian in metres; sh: degree of the spherical
    harmonics, -1 for flat colour; quartets: raw quads of one phase offset per
    frame, each at its own time; bg: random backgrounds."""
    c = dict(kind=kind, n=n, frames=frames, width=width, height=height, freqs=1, tile_w=16, tile_h=16,
             dynamic=frames > 1, quartets=False, sh=-1, size=0.03, bg=False)
    c.update(more)
    return c


def _net(kind, n, times):
    """A deformation-network case: "netfwd" (inference) or "netbwd" (training
    forward and backward) for n centres at the given number of times."""
    return dict(kind=kind, n=n, frames=times)


def listed():
    def named(name, c):
        return dict(c, name=name)

    return [
        # interactive editing or a unit test of a user's pipeline: a toy scene,
        # where the launches and the host call are what one waits for
        named("tiny_2k_64x48", _scene("fwdbwd", 2000, 1, 64, 48)),
        # the same through autograd, at an odd image size, with two modulation
        # frequencies, 8x8 tiles and a random background
        named("autograd_4k_97x75_2f", _scene("render", 4001, 2, 97, 75, freqs=2, tile_w=8, tile_h=8, bg=True)),
        # a viewer of a captured scene at the sensor resolution: forward only
        named("view_100k_320x240", _scene("view", 100_000, 1, 320, 240)),
        # single-frame fitting of a static scene at 640 x 480
        named("frame_100k_640x480", _scene("fwdbwd", 100_000, 1, 640, 480)),
        # a batch of frames of a dynamic scene, the usual training batch
        named("batch_200k_640x480_8f", _scene("fwdbwd", 200_000, 8, 640, 480)),
        # raw quads of asynchronous quartets, ragged count and image
        named("quartets_120k_500x375_8f", _scene("fwdbwd", 120_011, 8, 500, 375, quartets=True, bg=True)),
        # view-dependent colour and reflectivity (degree 3)
        named("harmonics_100k_640x480_4f", _scene("fwdbwd", 100_003, 4, 640, 480, sh=3)),
        # the largest scene: a million Gaussians, two frequencies
        named("large_1m_1024x768_16f", _scene("fwdbwd", 1_000_000, 16, 1024, 768, freqs=2)),
        # one optimisation step over a sequence (select, render, losses, backward, Adam)
        named("train_300k_640x480_b4", _scene("train", 300_000, 4, 640, 480, bg=True)),
        # the same with the deformation network in the captured step
        named("trainnet_100k_640x480_b4", _scene("trainnet", 100_000, 4, 640, 480, bg=True)),
        # the deformation network alone: a training batch, and a small inference
        named("net_train_200k_8t", _net("netbwd", 200_000, 8)),
        named("net_infer_20k_3t", _net("netfwd", 20_011, 3)),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["view", "fwdbwd", "fwdbwd", "fwdbwd", "render", "train", "trainnet", "netbwd", "netfwd"])
    if kind in ("netbwd", "netfwd"):
        times = rng.randint(1, 8)
        return _net(kind, int(_log(rng, 2000, 1_500_000 / times)), times)
    frames = int(_log(rng, 1, 16.99)) if kind in ("view", "fwdbwd", "render") else rng.randint(1, 4)
    height = int(_log(rng, 48, 768))
    width = int(height * rng.uniform(1.0, 4.0 / 3.0))
    # scenes hold up to about two Gaussians per pixel
    n = int(_log(rng, 2000, min(600_000, 3_000_000 / frames, 2 * width * height)))
    if kind == "trainnet":
        n = min(n, 200_000)
    # the footprint in pixels grows with the image (its focal length does), so
    # larger counts take smaller Gaussians, as reconstructions do
    size = 0.03 * rng.uniform(0.3, 1.1) * min(1.0, (200_000 / n) ** 0.25)
    tile_w, tile_h = rng.choice([(16, 16), (16, 16), (16, 16), (32, 8), (8, 8)])
    if tile_w == 8 and height > 320:
        tile_w = tile_h = 16
    quartets = kind in ("view", "fwdbwd") and rng.random() < 0.2
    sh = rng.choice([-1, -1, -1, 1, 2, 3])
    return _scene(kind, n, frames, width, height, freqs=rng.choice([1, 1, 2, 3, 4]) if not quartets else rng.choice([1, 2]),
                  tile_w=tile_w, tile_h=tile_h, dynamic=frames > 1 or rng.random() < 0.5, quartets=quartets,
                  sh=sh if kind != "view" or sh < 2 else -1, size=round(size, 5), bg=rng.random() < 0.5)


# ----------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------

def _focal(c):
    return 525.0 * c["width"] / 640.0


def _gaussians(c, g, dev):
    """float32 parameter tensors of a scene drawn from the generator g."""
    n, W, H, f = c["n"], c["width"], c["height"], _focal(c)

    def uni(*shape):
        return torch.rand(*shape, generator=g, device=dev)

    def nor(*shape):
        return torch.randn(*shape, generator=g, device=dev)

    z = 0.5 + 4.0 * uni(n)
    x = (uni(n) - 0.5) * W * z / f
    y = (uni(n) - 0.5) * H * z / f
    quat = nor(4, n)
    p = dict(mean=torch.stack([x, y, z]).contiguous(), vel=None, acc=None,
             scale=torch.exp(math.log(c["size"]) + 0.3 * nor(3, n)), quat=quat / quat.norm(dim=0),
             omega=None, opacity_logit=nor(n), rgb=uni(3, n), albedo=uni(n))
    if c["dynamic"]:
        p.update(vel=0.5 * nor(3, n), acc=nor(3, n), omega=nor(3, n))
    if c["sh"] >= 0:
        K = (c["sh"] + 1) ** 2
        fall = torch.tensor([0.3 / (l + 1) for l in range(c["sh"] + 1) for _ in range(2 * l + 1)], device=dev)
        y00 = 0.5 / math.sqrt(math.pi)
        sh_rgb = nor(K, 3, n) * fall[:, None, None]
        sh_alb = nor(K, n) * fall[:, None]
        sh_rgb[0] = (p["rgb"] - 0.5) / y00
        sh_alb[0] = (p["albedo"] - 0.5) / y00
        p.update(rgb=None, albedo=None, sh_rgb=sh_rgb.contiguous(), sh_albedo=sh_alb.contiguous())
    return p


def _config(c):
    return raster.RasterConfig(width=c["width"], height=c["height"], freqs=FREQS[:c["freqs"]], phases=PHASES,
                               tile_w=c["tile_w"], tile_h=c["tile_h"])


class _Frame:
    """A camera at the origin, as raster.pack_frames reads it."""

    def __init__(self, c, i, total, bg):
        self.R = [1, 0, 0, 0, 1, 0, 0, 0, 1]
        self.t = [0, 0, 0]
        self.fx = self.fy = _focal(c)
        self.cx, self.cy = 0.5 * c["width"], 0.5 * c["height"]
        self.bg_rgb, self.bg_quad = bg[:3], bg[3:]
        self.t_lo = self.t_hi = 0.0
        self.quad_mask = 0
        self.time = 0.25 * i / max(total - 1, 1)
        if c["quartets"]:   # raw quad j of quartet q, at (q + j / 4) / 30 s
            q, j = divmod(i, 4)
            self.time, self.t_lo, self.t_hi = (q + j / 4) / 30, q / 30, (q + 1) / 30
            self.quad_mask = sum(1 << (4 * k + j) for k in range(c["freqs"]))


def _frames(c, g, dev, total=None):
    total = c["frames"] if total is None else total
    nq = 4 * c["freqs"]
    bg = 2.0 * torch.rand(total, 3 + nq, generator=g, device=dev) - 1.0
    bg = (bg if c["bg"] else 0.0 * bg).tolist()
    return [_Frame(c, i, total, bg[i]) for i in range(total)]


def _upstream(c, g, dev):
    F, H, W = c["frames"], c["height"], c["width"]
    return [torch.randn(F, k, H, W, generator=g, device=dev) for k in (3, 4 * c["freqs"])] + \
        [torch.randn(F, H, W, generator=g, device=dev)]


def _net_weights(net, g, dev, head=0.02):
    """Xavier-normal layers; the head as after some training."""
    parts = []
    for l in range(9):
        i, o = (84 if l == 0 else 256), (3 if l == 8 else 256)
        std = head if l == 8 else math.sqrt(2.0 / (i + o))
        parts += [std * torch.randn(o * i, generator=g, device=dev), 0.02 * torch.randn(o, generator=g, device=dev)]
    w = torch.cat(parts).contiguous()
    assert w.numel() == net.n_params
    return w


def prepare(case, seed):
    dev = torch.device("cuda")
    c = dict(case)
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    if c["kind"] in ("netfwd", "netbwd"):
        n, T = c["n"], c["frames"]
        net = deform.DeformNet(n, T, time_scale=4.0, training=c["kind"] == "netbwd", device=dev)
        x0 = torch.rand(3, n, generator=g, device=dev) * torch.tensor([[4.5], [4.5], [4.0]], device=dev) + \
            torch.tensor([[-2.25], [-2.25], [0.5]], device=dev)
        return dict(c=c, net=net, w=_net_weights(net, g, dev), x0=x0.contiguous(),
                    times=[0.25 * t / max(T - 1, 1) for t in range(T)],
                    d_delta=torch.randn(T, 3, n, generator=g, device=dev),
                    out=torch.empty(T, 3, n, device=dev))
    cfg = _config(c)
    params = _gaussians(c, g, dev)
    if c["kind"] in ("train", "trainnet"):
        return _prepare_train(c, cfg, params, g, dev)
    fr = raster.pack_frames(_frames(c, g, dev), cfg, dev)
    s = dict(c=c, cfg=cfg, params=params, frames=fr, up=_upstream(c, g, dev),
             ws=raster.Workspace(c["n"], c["frames"], cfg, max_pairs=_pairs(c), device=dev))
    if c["kind"] == "render":
        for k, v in params.items():
            if v is not None:
                v.requires_grad_()
        return s
    channels = ("rgb", "quad", "depth") + (("phasor", "amplitude") if c["kind"] == "view" else ())
    # raw quartets write one phase offset's quads a frame; the others stay as they were allocated
    s["out"] = {k: v.zero_() for k, v in raster.alloc_outputs(c["frames"], cfg, dev, channels).items()}
    s["grads"] = {k: torch.empty_like(v) if v is not None else None for k, v in params.items()}
    raster.forward(params, fr, cfg, s["ws"], out=s["out"])   # sizes the pair capacity, as a program does once
    return s


def _footprint(c):
    """Mean squared standard deviation of a splat in pixels."""
    return (c["size"] * _focal(c)) ** 2 * 0.444 * 1.2 + 0.3


def _pairs(c):
    """A guess at the (tile, Gaussian) pairs; prepare's first forward corrects it."""
    r = 3.0 * math.sqrt(_footprint(c))
    per = (2 * r / c["tile_w"] + 1) * (2 * r / c["tile_h"] + 1)
    return int(1.3 * c["n"] * c["frames"] * min(per, c["width"] * c["height"] / (c["tile_w"] * c["tile_h"]))) + 65536


def _prepare_train(c, cfg, params, g, dev):
    """A sequence of frames whose targets a second scene renders, and a
    trainable scene late in its schedule (rates at a hundredth)."""
    S, b = 3 * c["frames"], c["frames"]
    frames = raster.pack_frames(_frames(c, g, dev, S), cfg, dev)
    truth = _gaussians(dict(c, dynamic=True), g, dev)
    ws = raster.Workspace(c["n"], b, cfg, max_pairs=_pairs(c), device=dev)
    rgb, quad = [], []
    for i in range(0, S, b):
        o = raster.forward(truth, frames[i:i + b].contiguous(), cfg, ws)
        rgb.append(o["rgb"])
        quad.append(o["quad"])
    del ws
    bg = None
    if c["bg"]:
        bg = 2.0 * torch.rand(16, b, 3 + 4 * c["freqs"], generator=g, device=dev) - 1.0
    net = w = None
    if c["kind"] == "trainnet":
        net = deform.DeformNet(c["n"], b, time_scale=4.0, device=dev)
        w = _net_weights(net, g, dev, head=1e-3)
    params = {k: v for k, v in params.items() if v is not None}
    # one stream for every trainer of the process: its steps follow one another
    stream = _STREAMS.setdefault(dev, torch.cuda.Stream(device=dev))
    t = step.TrainStep({k: params.get(k) for k in tuple(FIELDS) + ("sh_rgb", "sh_albedo")}, frames,
                       torch.cat(rgb), torch.cat(quad), cfg, batch=b, bg_table=bg, max_pairs=_pairs(c),
                       lrs={k: 0.01 * v for k, v in step.DEFAULT_LR.items()}, net=net, net_params=w,
                       net_lr=8e-6, net_lr_final=1.6e-6, stream=stream)
    t.size_workspace()
    t.capture()
    return dict(c=c, train=t)


# ----------------------------------------------------------------------------
# One pass
# ----------------------------------------------------------------------------

def run(s):
    kind = s["c"]["kind"]
    if kind == "netfwd":
        return s["net"].forward(s["w"], s["x0"], s["times"], save=False, out=s["out"])
    if kind == "netbwd":
        delta = s["net"].forward(s["w"], s["x0"], s["times"], out=s["out"])
        d_w, d_x0 = s["net"].backward(s["w"], s["x0"], s["times"], s["d_delta"])
        return dict(delta=delta, d_w=d_w, d_x0=d_x0)
    if kind in ("train", "trainnet"):
        t = s["train"]
        t.replay()
        r = dict(loss=t.loss, rgb=t.out["rgb"], quad=t.out["quad"],
                 grads={k: v for k, v in t.grads.items() if v is not None},
                 params={k: v for k, v in t.params.items() if v is not None},
                 v={k: v for k, v in t.v.items() if v is not None})
        if t.net is not None:
            r.update(delta=t.delta, net_grad=t.net_grad, net_params=t.net_params)
        return r
    params, frames, cfg, ws, up = s["params"], s["frames"], s["cfg"], s["ws"], s["up"]
    if kind == "render":
        o = raster.render(params, frames, cfg, ws)
        leaves = [v for v in params.values() if v is not None]
        grads = torch.autograd.grad([o["rgb"], o["quad"], o["depth"]], leaves, up)
        names = [k for k, v in params.items() if v is not None]
        return dict(out={k: o[k] for k in ("rgb", "quad", "depth", "T_final", "n_contrib")},
                    grads=dict(zip(names, grads)))
    raster.forward(params, frames, cfg, ws, out=s["out"], check=False)
    if kind == "view":
        return s["out"]
    g = raster.backward(params, frames, cfg, ws, s["out"], *up, want_bg=s["c"]["bg"], grads=s["grads"])
    return dict(out=s["out"], grads={k: v for k, v in g.items() if v is not None})


# ----------------------------------------------------------------------------
# What a pass cannot do without
# ----------------------------------------------------------------------------

def _param_floats(c):
    K = (c["sh"] + 1) ** 2 if c["sh"] >= 0 else 1
    return 11 + (9 if c["dynamic"] else 0) + 4 * K


def work(c):
    n, F = c["n"], c["frames"]
    net_flop = 962_048.0 * n * F
    net_w = 4.0 * (84 * 256 + 7 * 256 * 256 + 3 * 256 + 8 * 256 + 3)
    if c["kind"] == "netfwd":
        return dict(bytes=net_w + 12.0 * n + 12.0 * n * F, flops=net_flop)
    if c["kind"] == "netbwd":
        return dict(bytes=2 * net_w + 24.0 * n + 24.0 * n * F, flops=3 * net_flop)
    px = float(F * c["width"] * c["height"])
    nq = 1 if c["quartets"] else 4 * c["freqs"]
    # Gaussians over a pixel, of which about a hundred are seen before it is opaque
    over = n * math.pi * 9.0 * _footprint(c) / (c["width"] * c["height"])
    seen = px * min(over, 100.0)
    scene = 4.0 * n * _param_floats(c)
    images = 4.0 * px * (3 + nq + 1 + 2)
    fwd = seen * (12 + 12 + 4 * c["freqs"])
    bwd = seen * (12 + 73 + 14 * c["freqs"])
    if c["kind"] == "view":
        return dict(bytes=scene + images + 4.0 * px * 3 * c["freqs"], flops=fwd)
    ups = 4.0 * px * (3 + nq + 1 + 2)
    w = dict(bytes=2 * scene + images + ups, flops=fwd + bwd)
    if c["kind"] in ("train", "trainnet"):
        # the targets are read, and Adam reads and writes its moments and the parameters
        w["bytes"] += 4.0 * px * (3 + nq) + 6 * scene
    if c["kind"] == "trainnet":
        w["bytes"] += 8 * net_w
        w["flops"] += 3 * net_flop
    return w


# ----------------------------------------------------------------------------
# The same in 64 bits
# ----------------------------------------------------------------------------

def exact(case, seed):
    c = dict(case)
    if c["kind"] in ("netfwd", "netbwd"):
        return _exact_net(c, seed)
    if c["kind"] in ("train", "trainnet") or c["sh"] >= 0 or c["quartets"] or \
            c["n"] * c["frames"] * c["width"] * c["height"] > 150_000_000:
        return None
    return _exact_render(c, seed)


def _exact_net(c, seed):
    s = prepare(dict(c, kind="netfwd"), seed)
    n, T = c["n"], c["frames"]
    train = c["kind"] == "netbwd"
    sx = float(s["net"].cfg.pos_scale)
    layers, at, w = [], 0, s["w"].double()
    for l in range(9):
        i, o = (84 if l == 0 else 256), (3 if l == 8 else 256)
        layers.append((w[at:at + o * i].view(o, i), w[at + o * i:at + o * i + o]))
        at += o * i + o
    delta = torch.empty(T, 3, n, dtype=torch.float64, device=w.device)
    x = s["x0"].double() * sx

    def encode(p):   # blocks p, sin(2^k pi p), cos(2^k pi p)
        return torch.cat([p] + [f(2.0 ** k * math.pi * p) for k in range(10) for f in (torch.sin, torch.cos)])

    for t in range(T):
        tt = torch.full((1, 1), float(ctypes.c_float(s["times"][t]).value) * 4.0, dtype=torch.float64, device=w.device)
        for a in range(0, n, 65536):
            p = x[:, a:a + 65536]
            h = torch.cat([encode(p), encode(tt).expand(21, p.shape[1])])
            for l, (W, b) in enumerate(layers):
                h = W @ h + b[:, None]
                h = h if l == 8 else torch.relu(h)
            delta[t, :, a:a + 65536] = h
    if not train:
        return delta
    # the products run in 16 bits, so units within rounding of their ReLU's kink are decided
    # otherwise than in 64 bits, which alone moves the gradients by 4 to 15 percent: no value
    return dict(delta=delta, d_w=None, d_x0=None)


def _exact_render(c, seed):
    s = prepare(c, seed)
    dev, cfg, F = s["frames"].device, s["cfg"], c["frames"]
    W, H, TW, TH = c["width"], c["height"], c["tile_w"], c["tile_h"]
    p = {k: (v.detach().double().requires_grad_() if v is not None else None) for k, v in s["params"].items()}
    fr = s["frames"].double()
    ys, xs = torch.meshgrid(torch.arange(H, device=dev), torch.arange(W, device=dev), indexing="ij")
    xs, ys = xs.reshape(-1).double() + 0.5, ys.reshape(-1).double() + 0.5
    tx, ty = (xs / TW).floor(), (ys / TH).floor()
    nq = 4 * c["freqs"]
    outs = dict(rgb=[], quad=[], depth=[], T_final=[], phasor=[], amplitude=[])
    bgs, total = [], 0.0
    f32 = lambda v: float(ctypes.c_float(v).value)
    for i in range(F):
        t = fr[i, 16]
        bg = fr[i, 17:20 + nq].clone().requires_grad_()
        bgs.append(bg)
        m, q = p["mean"], p["quat"]
        if p["vel"] is not None:
            m = m + p["vel"] * t + 0.5 * p["acc"] * t * t
            o, q0 = p["omega"], p["quat"]
            dq = torch.stack([-(o * q0[1:]).sum(0), *(q0[0] * o + torch.linalg.cross(o, q0[1:], dim=0))])
            q = q0 + 0.5 * t * dq
        w, x, y, z = q
        M = torch.stack([w * w + x * x - y * y - z * z, 2 * (x * y - w * z), 2 * (x * z + w * y),
                         2 * (x * y + w * z), w * w - x * x + y * y - z * z, 2 * (y * z - w * x),
                         2 * (x * z - w * y), 2 * (y * z + w * x), w * w - x * x - y * y + z * z]).view(3, 3, -1)
        L = M * (p["scale"] / (q * q).sum(0))[None]
        fx, fy, cx, cy = fr[i, 12:16]
        X, Y, Z = m
        U = (fx / Z) * L[0] - (fx * X / Z / Z) * L[2]
        V = (fy / Z) * L[1] - (fy * Y / Z / Z) * L[2]
        dil = f32(cfg.dilation)
        a, b, d = (U * U).sum(0) + dil, (U * V).sum(0), (V * V).sum(0) + dil
        det = a * d - b * b
        u, v = fx * X / Z + cx, fy * Y / Z + cy
        R = m.norm(dim=0)
        with torch.no_grad():   # the tiles whose pixel centres meet the box of the 3 sigma ellipse
            ext = f32(cfg.extent_sigma)
            lo_x, hi_x = ((u - ext * a.sqrt() + 0.5) / TW).floor(), ((u + ext * a.sqrt() - 0.5) / TW).floor()
            lo_y, hi_y = ((v - ext * d.sqrt() + 0.5) / TH).floor(), ((v + ext * d.sqrt() - 0.5) / TH).floor()
            order = torch.argsort(Z.float(), stable=True)
            order = order[(Z > f32(cfg.near_z))[order]]
        k = order
        dx, dy = xs[:, None] - u[k], ys[:, None] - v[k]
        G = torch.exp(-0.5 * (d[k] * dx * dx - 2 * b[k] * dx * dy + a[k] * dy * dy) / det[k])
        al = torch.clamp(torch.sigmoid(p["opacity_logit"])[k] * G, max=f32(cfg.alpha_max))
        with torch.no_grad():
            on = (tx[:, None] >= lo_x[k]) & (tx[:, None] <= hi_x[k]) & (ty[:, None] >= lo_y[k]) & (ty[:, None] <= hi_y[k])
            on &= al >= f32(cfg.alpha_min)
            after = torch.cumprod(torch.where(on, 1 - al, torch.ones_like(al)), 1)
            on &= after >= f32(cfg.T_min)
        al = torch.where(on, al, torch.zeros_like(al))
        after = torch.cumprod(1 - al, 1)
        T = torch.cat([torch.ones_like(after[:, :1]), after[:, :-1]], 1)
        Tf = after[:, -1]
        w1 = al * T
        w2 = w1 * T
        rgb = torch.stack([w1 @ p["rgb"][ch][k] + bg[ch] * Tf for ch in range(3)])
        dep = w1 @ R[k]
        amp = cfg.source_intensity * p["albedo"] / (R * R)
        quad, pha = [], []
        for f in range(c["freqs"]):
            psi = 4 * math.pi * cfg.freqs[f] / LIGHT * R
            S, C = w2 @ (amp * torch.sin(psi))[k], w2 @ (amp * torch.cos(psi))[k]
            js = [math.cos(ph) * S + math.sin(ph) * C + bg[3 + 4 * f + j] * Tf for j, ph in enumerate(PHASES)]
            quad += js
            pha += [sum(math.sin(ph) * v for ph, v in zip(PHASES, js)), sum(math.cos(ph) * v for ph, v in zip(PHASES, js))]
        quad, pha = torch.stack(quad), torch.stack(pha)
        total = total + (rgb.view(3, H, W) * s["up"][0][i].double()).sum() + \
            (quad.view(nq, H, W) * s["up"][1][i].double()).sum() + (dep.view(H, W) * s["up"][2][i].double()).sum()
        keep = dict(rgb=rgb.view(3, H, W), quad=quad.view(nq, H, W), depth=dep.view(H, W), T_final=Tf.view(H, W),
                    phasor=pha.view(-1, 2, H, W), amplitude=0.5 * pha.view(-1, 2, H, W).norm(dim=1))
        for name, value in keep.items():
            outs[name].append(value.detach())
    outs = {k: torch.stack(v) for k, v in outs.items()}
    outs["n_contrib"] = None
    if c["kind"] == "view":
        return outs
    names = [k for k, v in p.items() if v is not None]
    grads = torch.autograd.grad(total, [p[k] for k in names] + bgs)
    g = dict(zip(names, grads))
    if c["kind"] == "fwdbwd" and c["bg"]:
        g["bg"] = torch.stack(grads[len(names):])
    return dict(out={k: outs[k] for k in ("rgb", "quad", "depth", "T_final", "n_contrib")}, grads=g)
