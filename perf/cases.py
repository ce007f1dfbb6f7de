"""Timed cases of the renderer: the calls its users make, over the sizes they make them at.

A case is a dict of plain values.  ``listed()`` names the fixed ones, ``draw(rng)``
gives one more of the same ranges, ``prepare(case, seed)`` makes what a program has
in hand before the call (scene, cameras, targets, the renderer with its fixed pair
capacity, Adam's moments), ``run(state)`` is one call, ``work(case)`` the bytes and
operations it cannot do without, and ``exact(case, seed)`` the same outputs in
float64 by plain torch: every Gaussian's slice and projection written from the
method, a per-tile depth-ordered list, and autograd.

Scenes follow the recipes of ``synth`` (noisy unit sphere, cube, and their mix),
drawn on the GPU.  Targets are smooth random images; the Adam moments are those of
a run under way (a thousand steps in) with the learning rates of its late phase, so
that repeated steps keep the scene what it is.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import synth
from paper_2410_04974_amd import Render6D, Renderer, Trainer
from paper_2410_04974_amd._lib import build_cache
from paper_2410_04974_amd.render import DEFAULT_LR

STEPS_TAKEN = 1000          # Adam steps behind a training state
LATE_LR = 0.01              # share of the initial learning rates
LAMBDA = 0.35               # the renderer's default directional-opacity strength
UNEVEN = ((400, 400), (800, 800), (1280, 720), (1600, 900))


def listed():
    return [
        # a preview or a unit of a test suite: launches and host work are all there is
        dict(name="render_1k_128", kind="render", n=1000, scene="cube", w=128, h=128, cached=False, fixed=False),
        # novel-view rendering of a trained volume (cloud, smoke): ~1e4 wide Gaussians, one large view
        dict(name="render_12k_1408_cached", kind="render", n=12657, scene="volume", w=1408, h=1408, cached=True,
             fixed=True),
        # novel-view rendering of a trained object: ~2e5 Gaussians
        dict(name="render_175k_1408_cached", kind="render", n=174746, scene="sphere", w=1408, h=1408, cached=True,
             fixed=True),
        # a training step early in a run (few Gaussians, a ragged small image)
        dict(name="train_20k_403x301", kind="train", n=20011, scene="cube", w=403, h=301, views=1),
        # the training step of a full scene, one 800x800 view: the benchmark's workload
        dict(name="train_300k_800", kind="train", n=300000, scene="inward", w=800, h=800, views=1),
        # the same with the full photometric loss, a learnable lambda and densification statistics
        dict(name="train_100k_801x599_full_loss", kind="train", n=100003, scene="sphere", w=801, h=599, views=1,
             dssim=0.2, learn_lambda=True, stats=True),
        # the colour ablation (one RGB triple per Gaussian) through the separate backward and Adam
        dict(name="train_50k_640x480_rgb_unfused", kind="train", n=50021, scene="sphere", w=640, h=480, views=2,
             rgb=True, fused=False),
        # a large scene, eight 1080p views a step, the step replayed from a captured graph
        dict(name="train_1m_8x1080p_graph", kind="train", n=1000000, scene="mixed", w=1920, h=1080, views=8,
             graph=True),
        # many uneven views rendered and differentiated in one call
        dict(name="views16_500k_fwd_bwd", kind="views", n=500000, scene="sphere", views=16, w=0, h=0),
        # the renderer inside a torch program: autograd with an upstream gradient
        dict(name="autograd_100k_800", kind="autograd", n=100000, scene="sphere", w=800, h=800),
        # clone / split / prune of a scene with its Adam moments
        dict(name="density_300k", kind="density", n=300000, scene="inward"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["render", "render", "train", "train", "train", "views", "autograd", "density"])
    scene = rng.choice(["cube", "sphere", "sphere", "inward", "mixed"])
    if kind == "render":
        return dict(kind=kind, n=log_int(300, 400000), scene=rng.choice(["cube", "sphere", "volume"]),
                    w=log_int(64, 1600), h=log_int(64, 1600), cached=rng.random() < 0.5, fixed=rng.random() < 0.6,
                    tile=rng.choice([16, 16, 8, 32]))
    if kind == "train":
        fused = rng.random() < 0.8
        return dict(kind=kind, n=log_int(1000, 400000), scene=scene, w=log_int(64, 1200), h=log_int(64, 1200),
                    views=rng.choice([1, 1, 1, 2, 3, 4]), dssim=rng.choice([0.0, 0.0, 0.2]),
                    learn_lambda=rng.random() < 0.3, stats=rng.random() < 0.5, rgb=rng.random() < 0.2, fused=fused,
                    graph=fused and rng.random() < 0.4)
    if kind == "views":
        return dict(kind=kind, n=log_int(1000, 300000), scene=scene, views=rng.randint(2, 16), w=log_int(64, 900),
                    h=log_int(64, 900))
    if kind == "autograd":
        return dict(kind=kind, n=log_int(1000, 300000), scene=scene, w=log_int(64, 1200), h=log_int(64, 1200))
    return dict(kind=kind, n=log_int(2000, 1000000), scene=scene)


# ------------------------------------------------------------------ inputs
def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 16 + stream)


def _scene(case, seed):
    """Raw parameters [76, n] by the recipe of synth.make_scene, drawn on the GPU."""
    n, kind = case["n"], case["scene"]
    g = _gen(seed, 0)

    def normal(mean, std, *shape):
        return mean + std * torch.randn(*shape, device="cuda", generator=g)

    def unit(k):
        v = normal(0.0, 1.0, 3, k)
        return v / v.norm(dim=0, keepdim=True)

    p = torch.empty((76, n), device="cuda")
    if kind in ("cube", "volume"):
        p[0:3] = torch.rand((3, n), device="cuda", generator=g) * 2 - 1
        p[3:6] = unit(n)
    else:
        nrm = unit(n)
        p[0:3] = nrm * (1 + normal(0.0, 0.05, n))
        if kind == "mixed":
            k = int(round(0.7 * n))
            p[0:3, k:] = torch.rand((3, n - k), device="cuda", generator=g) * 4 - 2
        p[3:6] = -nrm if kind == "inward" else unit(n)
    cross = 0.3 if kind == "inward" else 0.05
    spatial = -2.0 if kind == "volume" else -3.0
    direction = (-2.0, 0.5) if kind == "mixed" else (-1.0, 0.3)
    for k in range(21):
        if k in synth.DIAG_SPATIAL:
            m, s = spatial, 0.5
        elif k in synth.DIAG_DIRECTION:
            m, s = direction
        else:
            m, s = 0.0, cross if k in synth.CROSS_BLOCK else 0.05
        p[6 + k] = normal(m, s, n)
    p[27:75] = normal(0.0, 0.3, 48, n)
    p[75] = normal(-1.0 if kind == "volume" else 0.0, 1.0, n)
    return p


def _cameras(case, seed):
    """The views of a call: directions from the seed, sizes from the case."""
    k = case.get("views", 1)
    sizes = UNEVEN if case["w"] == 0 else [(case["w"], case["h"])]
    rng = np.random.default_rng(int(seed))
    cams = []
    for i in range(k):
        d = rng.normal(size=3)
        d[2] *= 0.6  # not along the up axis
        w, h = sizes[i % len(sizes)]
        cams.append(synth.look_at_camera(4.0 * d / np.linalg.norm(d), w, h))
    return cams


def _targets(case, seed, cams):
    """A smooth random image in (0, 1) per view."""
    g = _gen(seed, 1)
    out = []
    for c in cams:
        low = torch.rand((1, 3, 12, 12), device="cuda", generator=g)
        out.append(torch.nn.functional.interpolate(low, size=(c.height, c.width), mode="bilinear",
                                                   align_corners=False)[0].contiguous())
    return out


def _upstream(case, seed, cams):
    g = _gen(seed, 2)
    return [torch.randn((3, c.height, c.width), device="cuda", generator=g) for c in cams]


def _moments(case, seed, cams):
    """Adam moments of a run under way: gradients of a few image elements' weight."""
    g = _gen(seed, 3)
    s = 4.0 / sum(3 * c.width * c.height for c in cams)
    shape = (76, case["n"])
    m = torch.randn(shape, device="cuda", generator=g) * (0.3 * s)
    v = (torch.rand(shape, device="cuda", generator=g) + 0.5) * (s * s)
    return m, v


def _lambda_state(case, seed, cams):
    g = _gen(seed, 4)
    s = 4.0 / sum(3 * c.width * c.height for c in cams)
    n = case["n"]
    raw = torch.randn(n, device="cuda", generator=g) * 0.5 - 0.6
    m = torch.randn(n, device="cuda", generator=g) * (0.3 * s)
    v = (torch.rand(n, device="cuda", generator=g) + 0.5) * (s * s)
    return raw, m, v


def _density_inputs(case, seed):
    """A scene at a density-control step: a twentieth of its Gaussians faded out, a fifth of
    the others (one in 150 of these never seen) with a mean screen gradient over the 3DGS
    threshold 2e-4, the rest below it.  The shares are exact, so every seed gives the same counts."""
    n = case["n"]
    p = _scene(case, seed)
    g = _gen(seed, 5)
    perm = torch.randperm(n, device="cuda", generator=g)
    faded, grown = perm[:n // 20], perm[n // 20:n // 20 + n // 5]
    p[75].clamp_(min=-4.0)
    p[75, faded] = -6.0
    mean = torch.exp(torch.randn(n, device="cuda", generator=g) * 0.7 + math.log(4e-5)).clamp(max=1.8e-4)
    mean[grown] = 2.2e-4 * torch.exp(torch.rand(grown.numel(), device="cuda", generator=g) * 1.5)
    cnt = torch.randint(1, 65, (n,), device="cuda", generator=g).float()
    cnt[grown[::150]] = 0
    return p, torch.stack([mean * cnt, cnt]).contiguous()


def _fix_capacity(r, params, cams):
    """Grow on demand once, then a fixed pair capacity with half as much again (no host waits)."""
    r.forward(params, cams)
    r.configure(pair_capacity=int(r.ctx.sizes()["pairs"] * 1.5) + 4096)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "density":
        params, stats = _density_inputs(case, seed)
        g = _gen(seed, 6)
        m, v = _moments(case, seed, [synth.default_camera(800, 800)])
        return dict(kind=kind, r=Renderer(), params=params, m=m, v=v, stats=stats,
                    noise=torch.randn((2, 3, case["n"]), device="cuda", generator=g))
    params = _scene(case, seed)
    cams = _cameras(case, seed)
    tile = case.get("tile", 16)
    r = Renderer(tile=(tile, 256 // tile), rgb_color=case.get("rgb", False))
    st = dict(kind=kind, r=r, params=params, cams=cams)
    if kind == "render":
        if case["fixed"]:
            _fix_capacity(r, params, cams)
        st["cache"] = build_cache(params) if case["cached"] else None
        st["out"] = [torch.empty((3, c.height, c.width), device="cuda") for c in cams]
    elif kind == "views":
        _fix_capacity(r, params, cams)
        st["dl"] = _upstream(case, seed, cams)
        st["out"] = [torch.empty((3, c.height, c.width), device="cuda") for c in cams]
        st["grad"] = torch.empty_like(params)
    elif kind == "autograd":
        _fix_capacity(r, params, cams)
        st["params"] = params.requires_grad_(True)
        st["dl"] = _upstream(case, seed, cams)
    else:
        _fix_capacity(r, params, cams)
        raw = None
        if case.get("learn_lambda"):
            raw, ml, vl = _lambda_state(case, seed, cams)
        tr = Trainer(params, r, lr=tuple(LATE_LR * x for x in DEFAULT_LR), lambda_raw=raw, lr_lambda=LATE_LR * 1e-2,
                     lambda_dssim=case.get("dssim", 0.0))
        m, v = _moments(case, seed, cams)
        targets = _targets(case, seed, cams)
        stats = torch.zeros((2, case["n"]), device="cuda") if case.get("stats") else None
        if case.get("graph"):
            first = params.clone()
            tr.capture(cams, targets, densify=stats, warmup=1)
            tr.params.copy_(first)
            if stats is not None:
                stats.zero_()
            if raw is not None:
                tr.lambda_raw.copy_(_lambda_state(case, seed, cams)[0])
        tr.m.copy_(m)
        tr.v.copy_(v)
        if raw is not None:
            tr.m_lambda.copy_(ml)
            tr.v_lambda.copy_(vl)
        tr.step_count = STEPS_TAKEN
        tr.step_counter.fill_(STEPS_TAKEN)
        st.update(tr=tr, targets=targets, stats=stats, fused=case.get("fused", True), graph=case.get("graph", False))
    return st


def run(st):
    kind, r = st["kind"], st["r"]
    if kind == "render":
        if st["cache"] is not None:
            return r.forward_cached(st["params"], st["cache"], st["cams"], out=st["out"])
        return r.forward(st["params"], st["cams"], out=st["out"])
    if kind == "views":
        imgs = r.forward(st["params"], st["cams"], out=st["out"])
        return {"images": imgs, "grad": r.backward(st["params"], st["dl"], grad=st["grad"])}
    if kind == "autograd":
        imgs = Render6D.apply(st["params"], r, st["cams"])
        (grad,) = torch.autograd.grad(imgs, st["params"], st["dl"])
        return {"images": list(imgs), "grad": grad}
    if kind == "density":
        p, m, v, _ = r.ctx.densify(st["params"], st["stats"], st["noise"], extent=4.0, m=st["m"], v=st["v"])
        return {"params": p, "m": m, "v": v}
    tr = st["tr"]
    loss = tr.replay() if st["graph"] else tr.step(st["cams"], st["targets"], densify=st["stats"], fused=st["fused"])
    out = {"loss": loss, "params": tr.params, "m": tr.m, "v": tr.v}
    if not st["fused"]:
        out["grad"] = tr.grad
    if st["stats"] is not None:
        out["stats"] = st["stats"]
    if tr.lambda_raw is not None:
        out.update(lambda_raw=tr.lambda_raw, grad_lambda=tr.grad_lambda, m_lambda=tr.m_lambda, v_lambda=tr.v_lambda)
    return out


# Contributions of a pixel (Gaussians with alpha >= 1/255 in front of saturation),
# measured on the 300k-Gaussian sphere at 800x800; other scenes are taken alike.
TAKEN = 75
FWD_FLOPS, BWD_FLOPS = 22, 52  # per contribution: evaluate and blend; re-evaluate and differentiate


def work(case):
    n, kind = case["n"], case["kind"]
    if kind == "density":
        # stats, noise and the three arrays read, about as much written
        return {"bytes": 4.0 * n * (2 + 6 + 2 * 3 * 76), "flops": 600.0 * n}
    px = sum(c.width * c.height for c in _cameras(case, 0))
    if kind == "render":
        rows = 6 + 48 + 22 if case["cached"] else 76
        return {"bytes": 4.0 * (rows * n + 3 * px), "flops": float(FWD_FLOPS * TAKEN * px)}
    both = float((FWD_FLOPS + BWD_FLOPS) * TAKEN * px)
    if kind in ("views", "autograd"):  # parameters, upstream gradient; images, gradient
        return {"bytes": 4.0 * (2 * 76 * n + 6 * px), "flops": both}
    rows = 6 * 76 + (76 if not case.get("fused", True) else 0)  # parameters and moments in and out (and the gradient)
    rows += 7 if case.get("learn_lambda") else 0
    rows += 4 if case.get("stats") else 0
    return {"bytes": 4.0 * (rows * n + 3 * px), "flops": both}


# ------------------------------------------------------------- float64 results
def _dot(a, b):
    return (a * b).sum(-1)


def _static(p):
    """The direction-independent part of the slice, [n, ...] in float64."""
    n = p.shape[1]
    cols = {}
    for i in range(6):
        for j in range(i + 1):
            r = p[6 + synth.tri_index(i, j)]
            cols[i, j] = torch.exp(r) if i == j else 2 * torch.sigmoid(r) - 1
    zero = torch.zeros(n, dtype=p.dtype, device=p.device)
    L = torch.stack([torch.stack([cols.get((i, j), zero) for j in range(6)], -1) for i in range(6)], -2)
    S = (L.unsqueeze(2) * L.unsqueeze(1)).sum(-1)
    Sp, Spd, Sd = S[:, :3, :3], S[:, :3, 3:], S[:, 3:, 3:]
    c0 = torch.linalg.cross(Sd[:, 1], Sd[:, 2])
    c1 = torch.linalg.cross(Sd[:, 2], Sd[:, 0])
    c2 = torch.linalg.cross(Sd[:, 0], Sd[:, 1])
    A = torch.stack([c0, c1, c2], -1) / _dot(Sd[:, 0], c0)[:, None, None]
    K = (Spd.unsqueeze(-1) * A.unsqueeze(1)).sum(2)
    Sc = Sp - (K.unsqueeze(2) * Spd.unsqueeze(1)).sum(-1)
    return A, K, Sc


def _sh(d):
    x, y, z = d.unbind(-1)
    c = math.sqrt
    pi = math.pi
    one = torch.ones_like(x)
    return torch.stack([
        c(1 / (4 * pi)) * one,
        c(3 / (4 * pi)) * y, c(3 / (4 * pi)) * z, c(3 / (4 * pi)) * x,
        c(15 / (4 * pi)) * x * y, c(15 / (4 * pi)) * y * z, c(5 / (16 * pi)) * (3 * z * z - 1),
        c(15 / (4 * pi)) * x * z, c(15 / (16 * pi)) * (x * x - y * y),
        c(35 / (32 * pi)) * y * (3 * x * x - y * y), c(105 / (4 * pi)) * x * y * z,
        c(21 / (32 * pi)) * y * (5 * z * z - 1), c(7 / (16 * pi)) * z * (5 * z * z - 3),
        c(21 / (32 * pi)) * x * (5 * z * z - 1), c(105 / (16 * pi)) * z * (x * x - y * y),
        c(35 / (32 * pi)) * x * (x * x - 3 * y * y)], -1)


def _project(p, static, cam, lam, rgb):
    """Screen-space records of one view: (u, v, Qxx, Qxy, Qyy, alpha, r, g, b) [n, 9],
    depth, extents and which Gaussians are drawn."""
    A, K, Sc = static
    R = torch.tensor(np.asarray(cam.R), dtype=p.dtype, device=p.device)
    t = torch.tensor(np.asarray(cam.t), dtype=p.dtype, device=p.device)
    C = -(R * t[:, None]).sum(0)
    mu_p = p[0:3].T
    d = mu_p - C
    x = d / d.norm(dim=-1, keepdim=True) - p[3:6].T
    mu = mu_p + _dot(K, x.unsqueeze(1))
    D = _dot(x, _dot(A, x.unsqueeze(1)))
    ac = torch.sigmoid(p[75]) * torch.exp(-lam * D)
    s = mu - C
    s = s / s.norm(dim=-1, keepdim=True)
    q = _dot(R, mu.unsqueeze(1)) + t
    z = torch.where(q[:, 2] > 0.2, q[:, 2], torch.ones_like(q[:, 2]))
    limx, limy = 1.3 * 0.5 * cam.width / cam.fx, 1.3 * 0.5 * cam.height / cam.fy
    xt = torch.clamp(q[:, 0] / z, -limx, limx)
    yt = torch.clamp(q[:, 1] / z, -limy, limy)
    T0 = (cam.fx / z)[:, None] * R[0] - (cam.fx * xt / z)[:, None] * R[2]
    T1 = (cam.fy / z)[:, None] * R[1] - (cam.fy * yt / z)[:, None] * R[2]
    S0, S1 = _dot(Sc, T0.unsqueeze(1)), _dot(Sc, T1.unsqueeze(1))
    cxx, cxy, cyy = _dot(T0, S0) + 0.3, _dot(T0, S1), _dot(T1, S1) + 0.3
    det = cxx * cyy - cxy * cxy
    u, v = cam.fx * q[:, 0] / z + cam.cx, cam.fy * q[:, 1] / z + cam.cy
    if rgb:
        col = torch.sigmoid(p[27:30].T)
    else:
        col = torch.sigmoid((p[27:75].T.reshape(-1, 16, 3) * _sh(s).unsqueeze(-1)).sum(1))
    rec = torch.cat([torch.stack([u, v, cyy / det, -cxy / det, cxx / det, ac], -1), col], -1)
    with torch.no_grad():
        qmax = 2 * torch.log(torch.clamp(255 * ac, min=1.0))
        ext = torch.stack([torch.sqrt(qmax * cxx), torch.sqrt(qmax * cyy)], -1)
        drawn = (q[:, 2] > 0.2) & (det > 0) & (255 * ac >= 1)
    return rec, q[:, 2].detach(), ext, drawn


class _View:
    """Depth-ordered 16x16 tile lists of one view, and the walk over them."""

    SEG = 256                  # list positions per step of the walk
    CELLS = 24_000_000         # (pixel, position) cells held at once

    def __init__(self, rec, depth, ext, drawn, cam):
        self.rec, self.W, self.H = rec, cam.width, cam.height
        self.ntx, nty = (cam.width + 15) // 16, (cam.height + 15) // 16
        self.nt = self.ntx * nty
        lo = torch.floor((rec[:, :2] - ext) / 16).long()
        hi = torch.floor((rec[:, :2] + ext) / 16).long() + 1
        top = torch.tensor([self.ntx, nty], device=rec.device)
        lo, hi = torch.minimum(lo.clamp(min=0), top), torch.minimum(hi.clamp(min=0), top)
        size = hi - lo
        cnt = torch.where(drawn, size[:, 0] * size[:, 1], torch.zeros_like(size[:, 0]))
        self.visible = cnt > 0
        idx = torch.nonzero(self.visible).flatten()
        idx = idx[torch.argsort(depth[idx].float(), stable=True)]
        c = cnt[idx]
        ent = torch.repeat_interleave(idx, c)
        k = torch.arange(ent.numel(), device=rec.device) - torch.repeat_interleave(torch.cumsum(c, 0) - c, c)
        w = size[ent, 0]
        tile = (lo[ent, 1] + k // w) * self.ntx + lo[ent, 0] + k % w
        o = torch.argsort(tile, stable=True)
        self.ent = ent[o]
        self.len = torch.bincount(tile, minlength=self.nt)
        self.start = torch.cumsum(self.len, 0) - self.len

    def pixels(self, tiles):
        i = torch.arange(256, device=tiles.device)
        return (tiles[:, None] % self.ntx) * 16 + i % 16, (tiles[:, None] // self.ntx) * 16 + i // 16

    def gather(self, tiles, s, length):
        """Entries [nt, length] at list positions s.., and which of them exist (below ends)."""
        pos = s + torch.arange(length, device=tiles.device)
        ok = pos < self.ends[tiles][:, None]
        at = torch.where(ok, self.start[tiles][:, None] + pos, torch.zeros_like(pos))
        return self.ent[at], ok

    @staticmethod
    def weights(r, ok, px, py, T):
        """alpha (0 where not taken) and transmittance behind each position, [nt, L, 256]."""
        dx = px[:, None, :] + 0.5 - r[..., 0, None]
        dy = py[:, None, :] + 0.5 - r[..., 1, None]
        q = r[..., 2, None] * dx * dx + 2 * r[..., 3, None] * dx * dy + r[..., 4, None] * dy * dy
        raw = r[..., 5, None] * torch.exp(-0.5 * q)
        a = torch.where(ok[..., None] & (raw >= 1 / 255), torch.clamp(raw, max=0.99), torch.zeros_like(raw))
        behind = T[:, None, :] * torch.exp(torch.cumsum(torch.log1p(-a), 1))
        return a, behind

    def walk(self, bg):
        """Image [3, H, W]; keeps each tile's length up to its last contribution and the final T."""
        dev = self.rec.device
        self.ends = self.len.clone()
        used = torch.zeros_like(self.len)
        C = torch.zeros((self.nt, 256, 3), dtype=torch.float64, device=dev)
        Tf = torch.ones((self.nt, 256), dtype=torch.float64, device=dev)
        order = torch.argsort(self.len, descending=True)
        for block in order.split(max(1, self.CELLS // (256 * self.SEG))):
            live, s = block[self.len[block] > 0], 0
            T = torch.ones((live.numel(), 256), dtype=torch.float64, device=dev)
            done = torch.zeros_like(T, dtype=torch.bool)
            while live.numel():
                ent, ok = self.gather(live, s, self.SEG)
                r = self.rec[ent]
                px, py = self.pixels(live)
                a, behind = self.weights(r, ok, px, py, T)
                keep = (behind >= 1e-4) & ~done[:, None, :]
                front = torch.cat([T[:, None, :], behind[:, :-1]], 1)
                wgt = torch.where(keep, a * front, torch.zeros_like(a))
                C[live] += torch.matmul(wgt.transpose(1, 2), r[..., 6:9])
                took = (wgt > 0).any(-1)
                pos = torch.arange(1, self.SEG + 1, device=dev) + s
                used[live] = torch.maximum(used[live], (took * pos).amax(1))
                T = torch.where(keep, behind, T[:, None, :].expand_as(behind)).amin(1)
                done = done | (behind[:, -1] < 1e-4)
                Tf[live] = T
                s += self.SEG
                on = (self.len[live] > s) & ~done.all(1)
                live, T, done = live[on], T[on], done[on]
        self.ends = used
        img = C + Tf[..., None] * bg
        return self.to_image(img)

    def to_image(self, x):
        px, py = self.pixels(torch.arange(self.nt, device=x.device))
        inside = (px < self.W) & (py < self.H)
        out = torch.zeros((x.shape[-1], self.H, self.W), dtype=x.dtype, device=x.device)
        out[:, py[inside], px[inside]] = x[inside].T
        return out

    def backward(self, dimg):
        """dL/drec [n, 9] for a background of zero, over the lists cut at their last contribution."""
        dev = self.rec.device
        grad = torch.zeros_like(self.rec)
        order = torch.argsort(self.ends, descending=True)
        order = order[self.ends[order] > 0]
        lens = self.ends[order].tolist()
        i = 0
        while i < len(lens):
            m = max(1, self.CELLS // (256 * lens[i]))
            tiles = order[i:i + m]
            ent, ok = self.gather(tiles, 0, lens[i])
            px, py = self.pixels(tiles)
            inside = (px < self.W) & (py < self.H)
            d = dimg[:, py.clamp(max=self.H - 1), px.clamp(max=self.W - 1)] * inside
            with torch.enable_grad():
                r = self.rec[ent].requires_grad_(True)
                T = torch.ones((tiles.numel(), 256), dtype=torch.float64, device=dev)
                a, behind = self.weights(r, ok, px, py, T)
                front = torch.cat([T[:, None, :], behind[:, :-1]], 1)
                wgt = torch.where(behind >= 1e-4, a * front, torch.zeros_like(a))
                img = torch.matmul(wgt.transpose(1, 2), r[..., 6:9])
                (g,) = torch.autograd.grad(img, r, d.permute(1, 2, 0))
            grad.index_add_(0, ent.flatten(), (g * ok[..., None]).flatten(0, 1))
            i += m
        return grad


def _ssim_loss(x, y, lam):
    """The 3DGS loss over float64 views: (1 - lam) L1 + lam (1 - SSIM)."""
    w = torch.exp(-(torch.arange(11, dtype=torch.float64, device=x[0].device) - 5) ** 2 / 4.5)
    w = w / w.sum()

    def blur(t):
        t = torch.nn.functional.pad(t, (5, 5, 5, 5))
        t = sum(w[k] * t[:, k:t.shape[1] - 10 + k, :] for k in range(11))
        return sum(w[k] * t[:, :, k:t.shape[2] - 10 + k] for k in range(11))

    total = sum(t.numel() for t in x)
    l1, ss = 0.0, 0.0
    for a, b in zip(x, y):
        l1 = l1 + (a - b).abs().sum()
        ma, mb = blur(a), blur(b)
        va, vb, cab = blur(a * a) - ma * ma, blur(b * b) - mb * mb, blur(a * b) - ma * mb
        s = ((2 * ma * mb + 1e-4) * (2 * cab + 9e-4)) / ((ma * ma + mb * mb + 1e-4) * (va + vb + 9e-4))
        ss = ss + s.sum()
    return (1 - lam) * l1 / total + lam * (1 - ss / total)


def _adam(p, g, m, v, lr, t):
    m1 = 0.9 * m + 0.1 * g
    v1 = 0.999 * v + 0.001 * g * g
    p1 = p - lr * (m1 / (1 - 0.9 ** t)) / (torch.sqrt(v1 / (1 - 0.999 ** t)) + 1e-15)
    return p1, m1, v1


def _exact_density(case, seed):
    p, st = _density_inputs(case, seed)
    p = p.double()
    noise = torch.randn((2, 3, case["n"]), device="cuda", generator=_gen(seed, 6)).double()
    m, v = (x.double() for x in _moments(case, seed, [synth.default_camera(800, 800)]))
    cand = torch.nonzero((st[1] > 0) & (st[0] / st[1].clamp(min=1) >= 2e-4)).flatten()
    w, vec = torch.linalg.eigh(_static(p[:, cand])[2].cpu())
    S = torch.sqrt(w.flip(-1).clamp(min=0)).cuda()
    vec = vec.flip(-1).cuda()
    big = vec.gather(1, vec.abs().argmax(1, keepdim=True))
    vec = vec * torch.sign(big)
    R = torch.stack([vec[..., 0], vec[..., 1], torch.linalg.cross(vec[..., 0], vec[..., 1])], -1)
    outs = (torch.sigmoid(p[75]) >= 0.01).long()
    split = torch.zeros(case["n"], dtype=torch.bool, device="cuda")
    split[cand] = (S[:, 0] > 0.01 * 4.0) & (outs[cand] > 0)
    outs[cand] *= 2
    src = torch.repeat_interleave(torch.arange(case["n"], device="cuda"), outs)
    second = torch.arange(src.numel(), device="cuda") - (torch.cumsum(outs, 0) - outs)[src]
    po, mo, vo = p[:, src], m[:, src], v[:, src]
    fresh = split[src] | (second == 1)
    mo[:, fresh] = 0
    vo[:, fresh] = 0
    slot = torch.zeros(case["n"], dtype=torch.long, device="cuda")
    slot[cand] = torch.arange(cand.numel(), device="cuda")
    at = torch.nonzero(split[src]).flatten()
    k = slot[src[at]]
    zs = noise[second[at], :, src[at]]
    po[0:3, at] += _dot(R[k], (S[k] * zs).unsqueeze(1)).T
    for r in (0, 2, 5):
        po[6 + r, at] -= math.log(1.6)
    for r in (1, 3, 4):
        q = torch.tanh(0.5 * po[6 + r, at]) / 1.6
        po[6 + r, at] = torch.log((1 + q) / (1 - q))
    return {"params": po, "m": mo, "v": vo}


def exact(case, seed):
    kind = case["kind"]
    with torch.no_grad():
        if kind == "density":
            return _exact_density(case, seed)
        p = _scene(case, seed).double()
        cams = _cameras(case, seed)
        rgb = case.get("rgb", False)
        train = kind == "train"
        raw = _lambda_state(case, seed, cams)[0].double() if case.get("learn_lambda") else None
        lam = torch.sigmoid(raw) if raw is not None else LAMBDA
        bg = torch.zeros(3, dtype=torch.float64, device="cuda")
        static = _static(p)
        views, imgs = [], []
        for c in cams:
            view = _View(*_project(p, static, c, lam, rgb), c)
            imgs.append(view.walk(bg))
            views.append(view)
        del static
        if kind == "render":
            return imgs
        if train:
            tgt = [t.double() for t in _targets(case, seed, cams)]
            with torch.enable_grad():
                leaf = [i.detach().requires_grad_(True) for i in imgs]
                if case.get("dssim", 0.0) > 0:
                    loss = _ssim_loss(leaf, tgt, case["dssim"])
                else:
                    loss = sum((a - b).abs().sum() for a, b in zip(leaf, tgt)) / sum(t.numel() for t in tgt)
                dl = torch.autograd.grad(loss, leaf)
        else:
            dl = [d.double() for d in _upstream(case, seed, cams)]
        stats = torch.zeros((2, case["n"]), dtype=torch.float64, device="cuda")
        grad = torch.zeros_like(p)
        grad_raw = torch.zeros_like(raw) if raw is not None else None
        for c, view, d in zip(cams, views, dl):
            g = view.backward(d)
            stats[0] += torch.sqrt((g[:, 0] * c.width / 2) ** 2 + (g[:, 1] * c.height / 2) ** 2)
            stats[1] += view.visible
            with torch.enable_grad():
                q = p.detach().requires_grad_(True)
                ins = [q] + ([raw.detach().requires_grad_(True)] if raw is not None else [])
                rec = _project(q, _static(q), c, torch.sigmoid(ins[1]) if raw is not None else LAMBDA, rgb)[0]
                got = torch.autograd.grad(rec[view.visible], ins, g[view.visible])
            grad += got[0]
            if raw is not None:
                grad_raw += got[1]
        if not train:
            return {"images": imgs, "grad": grad}
        lr = torch.empty((76, 1), dtype=torch.float64, device="cuda")
        for group, (lo, hi) in enumerate(((0, 3), (3, 6), (6, 27), (27, 30), (30, 75), (75, 76))):
            lr[lo:hi] = LATE_LR * DEFAULT_LR[group]
        m, v = (x.double() for x in _moments(case, seed, cams))
        out = {"loss": loss.detach().reshape(1)}
        out["params"], out["m"], out["v"] = _adam(p, grad, m, v, lr, STEPS_TAKEN + 1)
        if not case.get("fused", True):
            out["grad"] = grad
        if case.get("stats"):
            out["stats"] = stats
        if raw is not None:
            _, ml, vl = (x.double() for x in _lambda_state(case, seed, cams))
            out["lambda_raw"], out["m_lambda"], out["v_lambda"] = _adam(raw, grad_raw, ml, vl, LATE_LR * 1e-2,
                                                                       STEPS_TAKEN + 1)
            out["grad_lambda"] = grad_raw
        return out
