"""The work that users of this library have it do, as timed cases.

Every case is one call (or the one batched call) of a public entry point of
`paper_2604_03748_amd.lnm`, on synthetic inputs of the shapes and value ranges
that the path meets: guiding-map marches, whole frames, network inference,
the channel adapters, fine-step reference lightmaps and training gradients.
`exact` evaluates the same definitions with plain torch in fp64.
"""
from __future__ import annotations

import math
from dataclasses import dataclass

import numpy as np
import torch

from paper_2604_03748_amd import lnm

PRECISIONS = {"fp32": lnm.FP32, "bf16": lnm.BF16, "fp8": lnm.FP8_E4M3}
SIGMA = 8.0      # extinction scale of the configured scenes
DEPTH_TAU, ERT_EPS = 0.1, 1e-6  # defaults of lnm.make_params
DEV = "cuda"


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # a preview of a small volume: the smallest march, where launches and host time count
        dict(name="march_small", kind="march", grids="32x32x32", views="64x64", step=2.0, ortho=True, bricks=False),
        # the marches of one serving batch: static grids with resident bricks, 64^3 to 256^3
        dict(name="march_serving", kind="march", grids="64x64x64 128x128x128 192x192x192 256x256x256",
             views="128x128 256x256 256x256 512x512", step=4.0, ortho=False, bricks=True),
        # the headline frame: march, network, shading, in each precision's configured size
        dict(name="frame_fp32", kind="frame", grids="128x128x128", views="256x256", step=4.0, ortho=False,
             bricks=False, levels=4, base=32, precision="fp32", lights=1),
        dict(name="frame_fp8_512", kind="frame", grids="128x128x128", views="512x512", step=4.0, ortho=False,
             bricks=False, levels=4, base=32, precision="fp8", lights=1),
        # the large moving scene: a new 256^3 grid for each 1024^2 frame
        dict(name="frame_bf16_1024", kind="frame", grids="256x256x256", views="1024x1024", step=4.0, ortho=False,
             bricks=False, levels=4, base=48, precision="bf16", lights=2),
        # the network alone: a small ragged batch with its logits, a serving batch, an evaluation set
        dict(name="infer_small", kind="infer", levels=3, base=16, precision="fp32", batch=2, height=40, width=72,
             logits=True),
        dict(name="infer_bf16_batch", kind="infer", levels=4, base=32, precision="bf16", batch=16, height=256,
             width=256, logits=False),
        dict(name="infer_fp32_eval", kind="infer", levels=4, base=32, precision="fp32", batch=8, height=256,
             width=256, logits=False),
        # the adapters in place of the plain head
        dict(name="adapters", kind="adapters", base=32, levels=4, precision="fp32", batch=1, height=256, width=256),
        # training targets of a scene
        dict(name="reference", kind="reference", grids="128x128x128", views="256x256", step=0.5, ortho=False),
        # one training batch at each of the two configured scales, the small one with the adapters trained too
        dict(name="train_headline", kind="train", levels=4, base=32, batch=8, height=256, width=256, adapters=False),
        dict(name="train_small_adapters", kind="train", levels=3, base=16, batch=12, height=64, width=64,
             adapters=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, lo, hi):
    n = _log(rng, lo, hi)
    if rng.random() < 0.5:
        return f"{n}x{n}x{n}"
    return "x".join(str(max(16, int(n * rng.uniform(0.6, 1.0)))) for _ in range(3))


def _net_size(rng, levels, lo, hi):
    d = 1 << (levels - 1)
    return tuple(max(d, _log(rng, lo, hi) // d * d) for _ in range(2))


def draw(rng):
    kind = rng.choice(["march", "frame", "frame", "infer", "infer", "adapters", "reference", "train"])
    if kind == "march":
        n = rng.choice([1, 1, 2, 3])
        return dict(kind=kind, grids=" ".join(_grid(rng, 32, 256) for _ in range(n)),
                    views=" ".join(f"{_log(rng, 64, 512)}x{_log(rng, 64, 512)}" for _ in range(n)),
                    step=rng.choice([2.0, 4.0, 4.0]), ortho=rng.random() < 0.3, bricks=rng.random() < 0.5)
    if kind == "frame":
        levels, base = rng.choice([(3, 16), (4, 32), (4, 32), (4, 48)])
        h, w = _net_size(rng, levels, 64, 768)
        return dict(kind=kind, grids=_grid(rng, 32, 256), views=f"{w}x{h}", step=rng.choice([2.0, 4.0, 4.0]),
                    ortho=rng.random() < 0.2, bricks=rng.random() < 0.3, levels=levels, base=base,
                    precision=rng.choice(["fp32", "bf16", "fp8"]), lights=rng.choice([1, 2, 4]))
    if kind == "infer":
        levels, base = rng.choice([(3, 16), (4, 32), (4, 32), (4, 48)])
        h, w = _net_size(rng, levels, 40, 512)
        batch = max(1, min(_log(rng, 1, 16), (1 << 20) // (h * w)))
        return dict(kind=kind, levels=levels, base=base, precision=rng.choice(["fp32", "bf16", "fp8"]), batch=batch,
                    height=h, width=w, logits=rng.random() < 0.25)
    if kind == "adapters":
        levels, base = rng.choice([(3, 16), (4, 32), (4, 48), (3, 64)])
        h, w = _net_size(rng, levels, 64, 512)
        return dict(kind=kind, levels=levels, base=base, precision=rng.choice(["fp32", "bf16"]),
                    batch=max(1, min(_log(rng, 1, 4), (1 << 18) // (h * w))), height=h, width=w)
    if kind == "reference":
        return dict(kind=kind, grids=_grid(rng, 32, 128), views=f"{_log(rng, 64, 256)}x{_log(rng, 64, 256)}",
                    step=rng.choice([0.5, 1.0]), ortho=rng.random() < 0.4)
    levels, base = rng.choice([(3, 16), (4, 32)])
    h, w = _net_size(rng, levels, 64, 256)
    return dict(kind=kind, levels=levels, base=base, batch=max(1, min(_log(rng, 2, 12), (1 << 19) // (h * w))),
                height=h, width=w, adapters=rng.random() < 0.4)


# ------------------------------------------------------------------ inputs
@dataclass
class Camera:
    projection: int
    eye: tuple
    target: tuple = (0.5, 0.5, 0.5)
    up: tuple = (0.0, 1.0, 0.0)
    fov_y_deg: float = 60.0
    ortho_half_extent: float = math.sqrt(3.0) / 2.0
    width: int = 64
    height: int = 64


def _dims(text):
    return [tuple(int(v) for v in t.split("x")) for t in text.split()]


def _volume(shape, seed):
    """Soft blobs with small-scale modulation on an [nz][ny][nx] grid."""
    r = np.random.default_rng([seed, 1])
    blobs = 24
    ax = [(torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) / n for n in shape]
    cen, rad, peak = r.random((blobs, 3)), 0.05 + 0.15 * r.random(blobs), 0.5 + 1.5 * r.random(blobs)
    rho = torch.zeros(shape, device=DEV, dtype=torch.float64)
    for c, s, p in zip(cen, rad, peak):
        g = [torch.exp(-(a - x) ** 2 / (2 * s * s)) for a, x in zip(ax, c)]
        rho += p * g[0][:, None, None] * g[1][None, :, None] * g[2][None, None, :]
    noise = torch.zeros_like(rho)
    for f, a in ((4, 1.0), (8, 0.5), (16, 0.25)):
        ph = r.random(3) * 2 * math.pi
        w = [torch.sin(2 * math.pi * f * x + q) for x, q in zip(ax, ph)]
        noise += a * w[0][:, None, None] * w[1][None, :, None] * w[2][None, None, :]
    return torch.clamp(rho * (1.0 + 0.3 * noise / 1.75), min=0.0).to(torch.float32).contiguous()


def _camera(case, k, w, h, seed):
    """At distance 2.5 from the centre, on an orbit about the vertical axis."""
    a = np.random.default_rng([seed, 2, k]).random() * 2 * math.pi
    eye = (0.5 + 2.5 * math.cos(a), 0.5 + 0.4 * math.sin(3 * a), 0.5 + 2.5 * math.sin(a))
    proj = lnm.ORTHOGRAPHIC if case.get("ortho") else lnm.PERSPECTIVE
    return Camera(proj, eye, width=w, height=h)


def _scenes(case, seed):
    grids, views = _dims(case["grids"]), _dims(case["views"])
    vols = [_volume(g, seed + 1000 * k) for k, g in enumerate(grids)]
    cams = [_camera(case, k, w, h, seed) for k, (w, h) in enumerate(views)]
    return vols, cams


def _lights(case, seed):
    r = np.random.default_rng([seed, 3])
    out = []
    for _ in range(case["lights"]):
        d = r.normal(size=3)
        out.append((tuple(float(x) for x in d / np.linalg.norm(d)), tuple(float(x) for x in 0.3 + 0.7 * r.random(3))))
    return out


def _guides(batch, h, w, seed):
    """Guiding maps (in-scatter, transmittance, depth) of smoke that covers part of the view."""
    r = np.random.default_rng([seed, 4])
    y = (torch.arange(h, device=DEV, dtype=torch.float64) + 0.5) / h
    x = (torch.arange(w, device=DEV, dtype=torch.float64) + 0.5) / w
    out = []
    for _ in range(batch):
        tau = torch.zeros((h, w), device=DEV, dtype=torch.float64)
        for cy, cx, s, p in zip(*(r.random((4, 12)))):
            cy, cx, s, p = 0.2 + 0.6 * cy, 0.2 + 0.6 * cx, 0.03 + 0.12 * s, 0.5 + 4 * p
            tau += p * torch.exp(-(y - cy) ** 2 / (2 * s * s))[:, None] * torch.exp(-(x - cx) ** 2 / (2 * s * s))[None]
        f = 2 * math.pi * (4 + 8 * r.random(2))
        tau *= 1.0 + 0.3 * torch.sin(f[0] * y)[:, None] * torch.sin(f[1] * x)[None]
        T = torch.exp(-tau)
        D = torch.where(tau > 0.05, 2.0 + torch.floor(32 * T) / 32, torch.zeros_like(T))
        out.append(torch.stack([(1 - T) * (0.6 + 0.8 * T + 0.3 * y[:, None]), T, D], dim=-1))
    return torch.stack(out).to(torch.float32).contiguous()


def _targets(guide, seed):
    """sRGB lightmaps in [0, 1]: smooth functions of the guiding map."""
    r = np.random.default_rng([seed, 5])
    L, T = guide[..., :1].double(), guide[..., 1:2].double()
    a, b = (torch.as_tensor(r.random(6), device=DEV) for _ in range(2))
    return torch.clamp((0.2 + 0.5 * a) * L + 0.2 * b * (1 - T), 0, 1).to(torch.float32).contiguous()


def _layers(levels, base):
    """(c_in, c_out, kernel) in the parameter vector's order."""
    w = [base << l for l in range(levels)]
    out, cin = [], 3
    for l in range(levels):
        out += [(cin, w[l], 3), (w[l], w[l], 3)]
        cin = w[l]
    for l in range(levels - 2, -1, -1):
        out += [(w[l] + w[l + 1], w[l], 3), (w[l], w[l], 3)]
    return out + [(base, 6, 1)]


def _net_params(levels, base, seed):
    r = np.random.default_rng([seed, 6])
    parts = []
    for ci, co, k in _layers(levels, base):
        parts += [r.normal(size=co * ci * k * k) * math.sqrt(2.0 / (ci * k * k)), 0.2 * r.random(co) - 0.1]
    return np.concatenate(parts).astype(np.float32)


ADAPTER_TENSORS = ("ln1_w", "ln1_b", "conv1_w", "conv1_b", "dw_w", "dw_b", "sca_w", "sca_b", "conv3_w", "conv3_b",
                   "beta", "ln2_w", "ln2_b", "conv4_w", "conv4_b", "conv5_w", "conv5_b", "gamma", "head_w", "head_b")


def _adapter_shapes(c):
    return [(c,), (c,), (2 * c, c), (2 * c,), (2 * c, 9), (2 * c,), (c, c), (c,), (c, c), (c,), (c,), (c,), (c,),
            (2 * c, c), (2 * c,), (c, c), (c,), (c,), (2, c), (2,)]


def _adapter_params(c, seed):
    r = np.random.default_rng([seed, 7])
    parts = []
    for _ in range(4):
        for name, shape in zip(ADAPTER_TENSORS, _adapter_shapes(c)):
            n = int(np.prod(shape))
            if len(shape) == 2:
                parts.append(r.normal(size=n) * math.sqrt(2.0 / shape[1]))
            elif name in ("ln1_w", "ln2_w"):
                parts.append(0.8 + 0.4 * r.random(n))
            elif name in ("beta", "gamma"):
                parts.append(r.random(n) - 0.5)
            else:
                parts.append(0.2 * r.random(n) - 0.1)
    return np.concatenate(parts).astype(np.float32)


def _net(ctx, case, seed, h, w):
    levels, base, prec = case["levels"], case["base"], case["precision"]
    params = _net_params(levels, base, seed)
    scales = None
    if prec == "fp8":  # calibrated maxima, rounded up to powers of two
        amax = lnm.Net(ctx, levels, base, params).calibrate_amax(_guides(1, h, w, seed + 77))
        scales = np.exp2(np.ceil(np.log2(np.maximum(amax, 1e-6)))).astype(np.float32)
    return lnm.Net(ctx, levels, base, params, precision=PRECISIONS[prec], act_scales=scales)


# ------------------------------------------------------------------ states and passes
def prepare(case, seed):
    ctx, kind = lnm.Context(0), case["kind"]
    s = dict(kind=kind, ctx=ctx)
    if kind == "march":
        vols, cams = _scenes(case, seed)
        prms = [lnm.make_params(case["step"], seed=seed + k, frame=k) for k in range(len(vols))]
        bricks = [ctx.make_bricks(v) for v in vols] if case["bricks"] else [None] * len(vols)
        need = max(ctx.march_workspace_bytes(v, SIGMA, c, p, b) for v, c, p, b in zip(vols, cams, prms, bricks))
        s.update(vols=vols, cams=cams, prms=prms, bricks=bricks, scales=[SIGMA] * len(vols),
                 ws=torch.empty(need, dtype=torch.uint8, device=DEV),
                 outs=[torch.empty((c.height, c.width, 3), device=DEV) for c in cams])
    elif kind == "frame":
        vols, cams = _scenes(case, seed)
        cam, vol = cams[0], vols[0]
        net = _net(ctx, case, seed, cam.height, cam.width)
        prm = lnm.make_params(case["step"], seed=seed)
        br = ctx.make_bricks(vol) if case["bricks"] else None
        s.update(net=net, vol=vol, cam=cam, prm=prm, bricks=br, lights=_lights(case, seed),
                 ws=net.frame_workspace(vol, SIGMA, cam, prm, br),
                 outs=[torch.empty((cam.height, cam.width, c), device=DEV) for c in (3, 6, 4)])
    elif kind == "infer":
        b, h, w = case["batch"], case["height"], case["width"]
        net = _net(ctx, case, seed, h, w)
        s.update(net=net, guide=_guides(b, h, w, seed), out=torch.empty((b, h, w, 6), device=DEV),
                 logits=torch.empty((b, h, w, 6), device=DEV) if case["logits"] else None, ws=net.workspace(b, h, w))
    elif kind == "adapters":
        b, h, w = case["batch"], case["height"], case["width"]
        ad = lnm.Adapters(_net(ctx, case, seed, h, w), _adapter_params(case["base"], seed))
        s.update(ad=ad, guide=_guides(b, h, w, seed), out=torch.empty((b, h, w, 6), device=DEV),
                 extra=torch.empty((b, h, w, 2), device=DEV), ws=ad.workspace(b, h, w))
    elif kind == "reference":
        vols, cams = _scenes(case, seed)
        s.update(vol=vols[0], cam=cams[0], step=case["step"],
                 out=torch.empty((cams[0].height, cams[0].width, 6), device=DEV))
    else:
        b, h, w = case["batch"], case["height"], case["width"]
        tr = lnm.Trainer(ctx, case["levels"], case["base"], _net_params(case["levels"], case["base"], seed))
        if case["adapters"]:
            tr.attach_adapters(_adapter_params(case["base"], seed))
        g = _guides(b, h, w, seed)
        tr.workspace(b, h, w)
        s.update(tr=tr, guide=g, target=_targets(g, seed), adapters=case["adapters"])
    return s


def run(s):
    kind = s["kind"]
    if kind == "march":
        if len(s["vols"]) == 1:
            return s["ctx"].march(s["vols"][0], SIGMA, s["cams"][0], s["prms"][0], out=s["outs"][0], workspace=s["ws"],
                                  bricks=s["bricks"][0])
        return s["ctx"].march_batch(s["vols"], s["scales"], s["cams"], s["prms"], outs=s["outs"], workspace=s["ws"],
                                    bricks=s["bricks"])
    if kind == "frame":
        return s["net"].frame(s["vol"], SIGMA, s["cam"], s["prm"], lights=s["lights"], guide=s["outs"][0],
                              lightmaps=s["outs"][1], rgba=s["outs"][2], workspace=s["ws"], bricks=s["bricks"])
    if kind == "infer":
        s["net"].infer(s["guide"], out=s["out"], logits=s["logits"], workspace=s["ws"])
        return [s["out"]] if s["logits"] is None else [s["out"], s["logits"]]
    if kind == "adapters":
        return s["ad"].infer(s["guide"], out=s["out"], extra=s["extra"], workspace=s["ws"])
    if kind == "reference":
        return s["ctx"].reference_lightmaps(s["vol"], SIGMA, s["cam"], step_voxels=s["step"], srgb=True, out=s["out"])
    loss, grad = s["tr"].grad(s["guide"], s["target"])
    return [loss, grad, s["tr"].adapter_grad()] if s["adapters"] else [loss, grad]


# ------------------------------------------------------------------ the work of a pass
def _net_flops(levels, base, batch, h, w):
    total = 0.0
    for i, (ci, co, k) in enumerate(_layers(levels, base)):
        lvl = min(i // 2, levels - 1) if i < 2 * levels else max(0, levels - 2 - (i - 2 * levels) // 2)
        total += 2.0 * batch * (h >> lvl) * (w >> lvl) * ci * co * k * k
    return total


def _net_bytes(levels, base, batch, h, w, es):
    return es * sum(ci * co * k * k for ci, co, k in _layers(levels, base)) + batch * h * w * (12 + 24)


def _adapter_flops(c, batch, h, w):
    return 2.0 * 4 * batch * h * w * (6 * c * c + 18 * c + 2 * c)


def _march_work(case):
    """Grid read, guide written; about a third of a view's rays cross smoke for
    half the grid's depth, each sample marching two lights for a third of it."""
    nbytes = flops = 0.0
    for g, (w, h) in zip(_dims(case["grids"]), _dims(case["views"])):
        n = max(g) / case["step"]
        nbytes += 4.0 * g[0] * g[1] * g[2] + 12.0 * w * h
        flops += 40.0 * (w * h / 3) * (n / 2) * (1 + 2 * n / 3)
    return nbytes, flops


def work(case):
    kind = case["kind"]
    if kind in ("march", "frame"):
        nbytes, flops = _march_work(case)
        if kind == "frame":
            w, h = _dims(case["views"])[0]
            es = {"fp32": 4, "bf16": 2, "fp8": 1}[case["precision"]]
            nbytes += _net_bytes(case["levels"], case["base"], 1, h, w, es) + 16.0 * w * h
            flops += _net_flops(case["levels"], case["base"], 1, h, w)
        return {"bytes": nbytes, "flops": flops}
    if kind == "reference":
        g, (w, h) = _dims(case["grids"])[0], _dims(case["views"])[0]
        n = max(g) / case["step"]
        return {"bytes": 4.0 * g[0] * g[1] * g[2] + 24.0 * w * h, "flops": 40.0 * (w * h / 3) * (n / 2) * (1 + 6 * n / 3)}
    b, h, w = case["batch"], case["height"], case["width"]
    flops = _net_flops(case["levels"], case["base"], b, h, w)
    if kind == "infer":
        es = {"fp32": 4, "bf16": 2, "fp8": 1}[case["precision"]]
        return {"bytes": _net_bytes(case["levels"], case["base"], b, h, w, es), "flops": flops}
    if kind == "adapters":
        return {"bytes": _net_bytes(case["levels"], case["base"], b, h, w, 4) + 8.0 * b * h * w,
                "flops": flops + _adapter_flops(case["base"], b, h, w)}
    if case["adapters"]:
        flops += _adapter_flops(case["base"], b, h, w)
    # weights read and gradients written; forward, data and weight gradients
    return {"bytes": 2.0 * _net_bytes(case["levels"], case["base"], b, h, w, 4), "flops": 3.0 * flops}


# ------------------------------------------------------------------ the same in 64 bits
def _basis(cam):
    f = np.asarray(cam.target, np.float32).astype(np.float64) - np.asarray(cam.eye, np.float32).astype(np.float64)
    f /= np.linalg.norm(f)
    r = np.cross(f, np.asarray(cam.up, np.float64))
    r /= np.linalg.norm(r)
    return f, r, np.cross(r, f)


def _rays(cam):
    W, H = cam.width, cam.height
    f, r, u = (torch.as_tensor(v, device=DEV) for v in _basis(cam))
    sx = 2 * (torch.arange(W, device=DEV, dtype=torch.float64) + 0.5) / W - 1
    sy = 1 - 2 * (torch.arange(H, device=DEV, dtype=torch.float64) + 0.5) / H
    a = (sx * (W / H))[None, :, None].expand(H, W, 1)
    b = sy[:, None, None].expand(H, W, 1)
    eye = torch.as_tensor(np.asarray(cam.eye, np.float32).astype(np.float64), device=DEV)
    if cam.projection == lnm.PERSPECTIVE:
        d = f + math.tan(math.radians(cam.fov_y_deg) / 2) * (a * r + b * u)
        return eye.expand(H * W, 3), (d / d.norm(dim=-1, keepdim=True)).reshape(-1, 3)
    e = float(np.float32(cam.ortho_half_extent))
    return (eye + e * (a * r + b * u)).reshape(-1, 3), f.expand(H * W, 3)


class _Field:
    """sigma(x): zero-border, cell-centred trilinear interpolation."""

    def __init__(self, rho):
        self.n = torch.tensor(rho.shape[::-1], device=DEV, dtype=torch.float64)  # x, y, z
        nz, ny, nx = rho.shape
        self.g = torch.zeros((nz + 3, ny + 3, nx + 3), device=DEV, dtype=torch.float64)
        self.g[1:nz + 1, 1:ny + 1, 1:nx + 1] = rho
        self.g = self.g.reshape(-1)
        self.sy, self.sz = nx + 3, (nx + 3) * (ny + 3)
        self.lo, self.hi = -0.5 / self.n, 1 + 0.5 / self.n

    def __call__(self, x):
        g = torch.minimum(torch.clamp(x * self.n - 0.5, min=-1.0), self.n)
        i = torch.floor(g)
        f = g - i
        i = i.long() + 1
        at = i[:, 2] * self.sz + i[:, 1] * self.sy + i[:, 0]
        v = 0.0
        for dz in (0, 1):
            for dy in (0, 1):
                o = at + dz * self.sz + dy * self.sy
                row = self.g[o] * (1 - f[:, 0]) + self.g[o + 1] * f[:, 0]
                v = v + row * (f[:, 1] if dy else 1 - f[:, 1]) * (f[:, 2] if dz else 1 - f[:, 2])
        return SIGMA * v

    def clip(self, o, d):
        ta, tb = (self.lo - o) / d, (self.hi - o) / d
        flat = d == 0
        out = flat & ((o < self.lo) | (o > self.hi))
        inf = torch.full_like(ta, math.inf)
        a = torch.where(flat, -inf, torch.minimum(ta, tb)).amax(dim=1).clamp(min=0)
        b = torch.where(flat, inf, torch.maximum(ta, tb)).amin(dim=1)
        return a, torch.where(out.any(dim=1), torch.full_like(b, -1.0), b)

    def transmittance(self, x, l, h, tau_max):
        """From the points x toward l (one direction, or one each)."""
        l = l.expand_as(x)
        _, end = self.clip(x, l)
        steps = torch.floor(end / h).clamp(min=0)
        tau = torch.zeros_like(end)
        live = torch.nonzero(steps >= 1)[:, 0]
        k = 0
        while live.numel():
            k += 1
            s = self(x[live] + (k * h) * l[live]) * h
            tau[live] += s
            if k % 4 == 0:
                live = live[(steps[live] > k) & (tau[live] <= tau_max)]
            else:
                live = live[steps[live] > k]
        return torch.where(tau > tau_max, torch.zeros_like(tau), torch.exp(-tau))


def _jitter(seed, frame, n):
    with np.errstate(over="ignore"):
        z = (np.uint64(seed & (2**64 - 1)) ^ (np.uint64(frame) << np.uint64(32)) ^ np.arange(n, dtype=np.uint64))
        z = z + np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    return torch.as_tensor((z >> np.uint64(40)).astype(np.float64) / 2.0**24, device=DEV)


def _primary(field, o, d, h, u, tau_max, depth_tau):
    """Samples of the view rays: (pixel, t, weight, T before) of each, T and D per pixel."""
    t0, t1 = field.clip(o, d)
    n = torch.clamp(torch.ceil(t0 / h - u), min=1)
    n1 = torch.floor(t1 / h - u)
    P = o.shape[0]
    tau = torch.zeros(P, device=DEV, dtype=torch.float64)
    depth = torch.zeros_like(tau)
    rec = []
    live = torch.nonzero(n <= n1)[:, 0]
    while live.numel():
        t = (n[live] + u[live]) * h
        sig = field(o[live] + t[:, None] * d[live])
        before = torch.exp(-tau[live])
        hit = (sig > depth_tau) & (depth[live] == 0)
        depth[live] = torch.where(hit, n[live] * h, depth[live])
        alpha = -torch.expm1(-sig * h)
        tau[live] += sig * h
        keep = alpha > 0
        rec.append((live[keep], t[keep], (before * alpha)[keep], before[keep]))
        n[live] += 1
        live = live[(n[live] <= n1[live]) & (tau[live] <= tau_max)]
    cat = [torch.cat(v) if rec else torch.zeros(0, device=DEV) for v in zip(*rec)] if rec else None
    return cat, torch.where(tau > tau_max, torch.zeros_like(tau), torch.exp(-tau)), depth


CHUNK = 1 << 21


def _exact_guide(rho, cam, step, seed, frame):
    field, (o, d) = _Field(rho), _rays(cam)
    h, tau_max = step / max(rho.shape), -math.log(ERT_EPS)
    rec, T, D = _primary(field, o, d, h, _jitter(seed, frame, o.shape[0]), tau_max, DEPTH_TAU)
    L = torch.zeros_like(T)
    if rec is not None:
        for lo in range(0, rec[0].numel(), CHUNK):
            p, t, A, before = (v[lo:lo + CHUNK] for v in rec)
            x, w = o[p] + t[:, None] * d[p], -d[p]
            top = torch.stack([w[:, 1], -w[:, 0], torch.zeros_like(w[:, 0])], dim=1)
            top = top / top.norm(dim=1, keepdim=True)
            v = before + field.transmittance(x, top, h, tau_max) + field.transmittance(x, -top, h, tau_max)
            L.index_add_(0, p, A * v)
    return torch.stack([L, T, D], dim=-1).reshape(cam.height, cam.width, 3)


def _exact_reference(rho, cam, step):
    field, (o, d) = _Field(rho), _rays(cam)
    h, tau_max = step / max(rho.shape), -math.log(ERT_EPS)
    rec, _, _ = _primary(field, o, d, h, torch.zeros(o.shape[0], device=DEV, dtype=torch.float64), tau_max, 0.0)
    f, r, u = _basis(cam)
    out = torch.zeros((o.shape[0], 6), device=DEV, dtype=torch.float64)
    if rec is not None:
        for a, ax in enumerate((r, -r, u, -u, -f, f)):
            l = torch.as_tensor(ax, device=DEV)
            for lo in range(0, rec[0].numel(), CHUNK):
                p, t, A, _ = (v[lo:lo + CHUNK] for v in rec)
                out[:, a].index_add_(0, p, A * field.transmittance(o[p] + t[:, None] * d[p], l, h, tau_max))
    out = torch.where(out <= 0.0031308, 12.92 * out, 1.055 * out.clamp(min=0) ** (1 / 2.4) - 0.055)
    return out.reshape(cam.height, cam.width, 6)


def _split(flat, shapes):
    out, at = [], 0
    for s in shapes:
        n = int(np.prod(s))
        out.append(flat[at:at + n].reshape(s))
        at += n
    return out


def _shifted(x, dy, dx):
    """x[b][y + dy][x + dx][c], zero outside."""
    B, H, W, C = x.shape
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    return p[:, 1 + dy:1 + dy + H, 1 + dx:1 + dx + W]


def _conv(x, w, b):
    B, H, W, C = x.shape
    y = b
    for t in range(9):
        y = y + _shifted(x, t // 3 - 1, t % 3 - 1).reshape(-1, C) @ w[:, :, t].t()
    return torch.relu(y).reshape(B, H, W, -1)


def _features(levels, base, flat, x):
    shapes = [s for ci, co, k in _layers(levels, base) for s in ((co, ci, k * k), (co,))]
    prm = _split(flat, shapes)
    it = iter(range(0, len(prm), 2))
    conv = lambda v: (lambda i: _conv(v, prm[i], prm[i + 1]))(next(it))  # noqa: E731
    skips = []
    for l in range(levels):
        if l:
            B, H, W, C = x.shape
            x = x.reshape(B, H // 2, 2, W // 2, 2, C).amax(dim=(2, 4))
        x = conv(conv(x))
        skips.append(x)
    for l in range(levels - 2, -1, -1):
        x = torch.cat([skips[l], x.repeat_interleave(2, dim=1).repeat_interleave(2, dim=2)], dim=-1)
        x = conv(conv(x))
    return x, prm[-2][:, :, 0], prm[-1]


def _naf(c, flat, x):
    """One adapter: the block and its head, sigmoid applied."""
    p = dict(zip(ADAPTER_TENSORS, _split(flat, _adapter_shapes(c))))
    norm = lambda v, k: torch.nn.functional.layer_norm(v, (c,), p[k + "_w"], p[k + "_b"], 1e-6)  # noqa: E731
    y = norm(x, "ln1") @ p["conv1_w"].t() + p["conv1_b"]
    d = p["dw_b"]
    for t in range(9):
        d = d + _shifted(y, t // 3 - 1, t % 3 - 1) * p["dw_w"][:, t]
    v = d[..., :c] * d[..., c:]
    v = v * (v.mean(dim=(1, 2), keepdim=True) @ p["sca_w"].t() + p["sca_b"])
    y = x + p["beta"] * (v @ p["conv3_w"].t() + p["conv3_b"])
    z = norm(y, "ln2") @ p["conv4_w"].t() + p["conv4_b"]
    z = (z[..., :c] * z[..., c:]) @ p["conv5_w"].t() + p["conv5_b"]
    return torch.sigmoid((y + p["gamma"] * z) @ p["head_w"].t() + p["head_b"])


def _adapted(c, flat, x):
    one = sum(int(np.prod(s)) for s in _adapter_shapes(c))
    fb, lr, ud, ae = (_naf(c, flat[k * one:(k + 1) * one], x) for k in range(4))
    return torch.cat([lr, ud, fb], dim=-1), ae


def _f64(a):
    return torch.as_tensor(np.asarray(a, np.float64), device=DEV)


def _exact_lightmaps(case, seed, guide):
    x, w, b = _features(case["levels"], case["base"], _f64(_net_params(case["levels"], case["base"], seed)), guide)
    z = x @ w.t() + b
    return torch.sigmoid(z), z


def _exact_shading(cam, lights, lm, guide):
    lin = torch.where(lm <= 0.04045, lm / 12.92, ((lm + 0.055) / 1.055) ** 2.4)
    f, r, u = _basis(cam)
    rgb = torch.zeros(lm.shape[:-1] + (3,), device=DEV, dtype=torch.float64)
    for d, col in lights:
        l = [float(np.dot(np.asarray(d, np.float64), v)) for v in (r, u, -f)]
        s = sum(abs(c) * lin[..., 2 * a + (c < 0)] for a, c in enumerate(l))
        rgb += s[..., None] * _f64(col)
    return torch.cat([rgb, 1 - guide[..., 1:2]], dim=-1)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("march", "frame", "reference"):
        vols, cams = _scenes(case, seed)
    if kind == "march":
        out = [_exact_guide(v, c, case["step"], seed + k, k) for k, (v, c) in enumerate(zip(vols, cams))]
        return out if len(out) > 1 else out[0]
    if kind == "reference":
        return _exact_reference(vols[0], cams[0], case["step"])
    if kind == "frame":
        g = _exact_guide(vols[0], cams[0], case["step"], seed, 0)
        if _net_flops(case["levels"], case["base"], 1, cams[0].height, cams[0].width) > 2.5e11:
            return [g, None, None]  # the 64-bit network would take too long
        lm = _exact_lightmaps(case, seed, g[None])[0][0]
        return [g, lm, _exact_shading(cams[0], _lights(case, seed), lm, g)]
    b, h, w = case["batch"], case["height"], case["width"]
    guide = _guides(b, h, w, seed)
    levels, base = case["levels"], case["base"]
    if kind == "infer":
        parts = [_exact_lightmaps(case, seed, guide[k:k + 1].double()) for k in range(b)]
        lm, z = (torch.cat(v) for v in zip(*parts))
        return [lm, z] if case["logits"] else [lm]
    if kind == "adapters":
        flat = _f64(_adapter_params(base, seed))
        x, _, _ = _features(levels, base, _f64(_net_params(levels, base, seed)), guide.double())
        return _adapted(base, flat, x)
    target = _targets(guide, seed).double()
    flat = _f64(_net_params(levels, base, seed)).requires_grad_()
    ad = _f64(_adapter_params(base, seed)).requires_grad_() if case["adapters"] else None
    loss = torch.zeros(1, device=DEV, dtype=torch.float64)
    for k in range(b):  # image by image: the loss is a mean over all of them
        x, hw, hb = _features(levels, base, flat, guide[k:k + 1].double())
        y = _adapted(base, ad, x)[0] if ad is not None else torch.sigmoid(x @ hw.t() + hb)
        part = ((y - target[k:k + 1]) ** 2).sum() / (b * h * w * 6)
        part.backward()
        loss += part.detach()
    return [loss, flat.grad] if ad is None else [loss, flat.grad, ad.grad]
