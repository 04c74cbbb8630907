"""The work this ray marcher is used for, as measurable cases.

Four kinds of use, each through the package's public entry points:

  train   one training step on full frames: culling build, forward, the
          gradient of a mean squared error, backward (payload and pose
          gradients), as ``bench.py`` steps it
  rays    the same step on a sampled subset of the pixels (Sec. 3.3)
  frame   one novel-view frame: culling build and forward only
  serve   a burst of requests to the serving scheduler on resident scenes

Scenes are synthetic, with the distributions of
``paper_2103_01954_amd/scenes.py`` (primitives on a noisy sphere or in a box,
random payloads with a share of empty voxels, cameras on a sphere of radius 3
looking at the centre), drawn on the GPU from the seed.  A case is a dict:

  kind, n primitives of m^3 voxels, bf16 payload or not, views of
  width x height, steps (samples per unit length, a power of two), fade (the
  opacity fade window of Sec. 3.1.3, 0: off), combine ("sum" or
  "sequential"), bg (composited over a background), empty (share of empty
  voxels), rays (sampled pixels of a "rays" case, else 0), requests (of a
  "serve" case, else 0)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2103_01954_amd.api import Context, DevicePrims, render
from paper_2103_01954_amd.scenes import SERVE_RESOLUTIONS, Camera, MarchParams
from paper_2103_01954_amd.serve import Server

DEV = "cuda"
EPS = 1e-6
POSE = ("pos", "rot", "scale")

_CTX = None


def _context():
    """A program keeps one context for its lifetime."""
    global _CTX
    if _CTX is None:
        _CTX = Context(0)
    return _CTX


# ----------------------------------------------------------------------------
# cases
# ----------------------------------------------------------------------------

def _case(kind, n, m, width, height, **kw):
    c = {"kind": kind, "n": n, "m": m, "bf16": False, "views": 1, "width": width, "height": height, "steps": 512,
         "fade": 0.0, "combine": "sum", "bg": False, "empty": 0.7, "rays": 0, "requests": 0}
    c.update(kw)
    return c


def listed():
    named = {
        # the smallest step: 8 boxes, 64 x 64, through the autograd function (unit
        # tests, smoke runs, fitting a few boxes): latency and launches
        "train_8x8_64": _case("train", 8, 8, 64, 64, steps=128, empty=0.0),
        # the smallest serving frame: a thumbnail of a BF16 scene of 16^3 payloads
        "frame_512x16_256_bf16": _case("frame", 512, 16, 256, 256, bf16=True),
        # many small primitives in a small picture: long culling lists
        "frame_16384x8_512_bf16": _case("frame", 16384, 8, 512, 512, bf16=True),
        # the 2M-voxel model rendered at one 1024^2 view
        "frame_4096x8_1024": _case("frame", 4096, 8, 1024, 1024),
        # a full-HD view of a BF16 scene with 12^3 payloads (height no multiple of a tile)
        "frame_2048x12_1080_bf16": _case("frame", 2048, 12, 1920, 1080, bf16=True),
        # the training mode on sampled rays, fade window and background as in the paper
        "rays_4096x8_4x4096": _case("rays", 4096, 8, 1024, 1024, views=4, rays=16384, fade=8.0, bg=True),
        # one ragged capture view (667 x 1024, the capture's frame) of the fade + background step
        "train_4096x8_667_fade_bg": _case("train", 4096, 8, 667, 1024, fade=8.0, bg=True),
        # the same voxel budget in fewer, larger primitives, traversal-order combine
        "train_512x16_667_seq": _case("train", 512, 16, 667, 1024, combine="sequential"),
        # ... and in the fewest the paper's ablation renders well: payloads of 32^3
        "train_64x32_667": _case("train", 64, 32, 667, 1024, steps=256),
        # the benchmark step: 4 views of 1024^2
        "train_4096x8_4x1024": _case("train", 4096, 8, 1024, 1024, views=4),
        # the large step: 32768 BF16 primitives of 16^3, 2 views of 2048^2
        "train_32768x16_2x2048_bf16": _case("train", 32768, 16, 2048, 2048, bf16=True, views=2, steps=1024, empty=0.8),
        # a burst of requests of the serving mix on four resident scenes
        "serve_16_requests": _case("serve", 4096, 12, 1920, 1080, bf16=True, requests=16),
    }
    return [dict(c, name=k) for k, c in named.items()]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    while True:
        kind = rng.choice(["train", "train", "rays", "frame", "frame", "serve"])
        m = rng.choice([4, 6, 8, 8, 8, 10, 12, 12, 16, 16, 24, 32])
        n = int(round(_log(rng, 8, 32768)))
        width, height = int(round(_log(rng, 64, 2048))), int(round(_log(rng, 64, 2048)))
        if max(width, height) > 3 * min(width, height):
            continue
        c = _case(kind, n, m, width, height, bf16=rng.random() < 0.5, views=rng.choice([1, 1, 1, 2, 3, 4]),
                  steps=rng.choice([128, 256, 512, 512, 1024]), fade=rng.choice([0.0, 0.0, 8.0]),
                  combine=rng.choice(["sum", "sum", "sum", "sequential"]), bg=rng.random() < 0.33,
                  empty=rng.choice([0.0, 0.5, 0.7, 0.8]))
        if kind == "rays":
            c["rays"] = min(c["views"] * width * height // 4, int(round(_log(rng, 1000, 65536))))
        if kind == "frame":
            c["views"] = 1
        if kind == "serve":
            c.update(bf16=True, views=1, fade=0.0, combine="sum", bg=False, requests=rng.randint(4, 16),
                     n=min(c["n"], 4096), m=min(m, 16), steps=512)
        if n * m ** 3 <= 134e6 and 1e3 <= _prim_samples(c) <= 0.8e9:
            return c


def _extent(c):
    """Half extent of a primitive: the shell stays covered as the number of primitives changes."""
    return min(0.4, 0.05 * math.sqrt(4096.0 / c["n"])) if not _boxes(c) else 0.25


def _boxes(c):
    return c["n"] < 32


def _prim_samples(c):
    """Expected (sample, primitive) pairs of one pass, from the boxes' volume and the ray density there."""
    vol = c["n"] * 8.0 * _extent(c) ** 3
    if c["kind"] == "serve":
        mean = sum(w * w for w, _ in SERVE_RESOLUTIONS) / len(SERVE_RESOLUTIONS)
        return c["requests"] * vol * mean / 9.0 * c["steps"]
    full = c["views"] * vol * c["width"] ** 2 / 9.0 * c["steps"]
    return full * (c["rays"] / (c["views"] * c["width"] * c["height"]) if c["rays"] else 1.0)


def work(case):
    c = case
    px = c["rays"] or c["views"] * c["width"] * c["height"]
    if c["kind"] == "serve":
        px = c["requests"] * sum(w * h for w, h in SERVE_RESOLUTIONS) / len(SERVE_RESOLUTIONS)
    scenes = 4 if c["kind"] == "serve" else 1
    payload = scenes * c["n"] * c["m"] ** 3 * 4
    back = c["kind"] in ("train", "rays")
    b = payload * (2 if c["bf16"] else 4) + c["n"] * 60 * scenes + px * 16 + (px * 12 if c["bg"] else 0)
    # forward: locate the cell, 8 weights, 4 channels of 8 corners, the sum
    f = _prim_samples(c) * 100
    if back:   # target in; payload and pose gradients out
        b += px * 12 + payload * 4 + c["n"] * 60 + (px * 12 if c["bg"] else 0)
        f += _prim_samples(c) * 150
    return {"bytes": float(b), "flops": float(f)}


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------

def _scene(c, gen):
    """{pos, rot, scale, payload} of a case as float32 tensors (payload bf16 if asked)."""
    n, m = c["n"], c["m"]
    f64 = dict(dtype=torch.float64, device=DEV, generator=gen)
    q = torch.randn(n, 4, **f64)
    if _boxes(c):
        pos = torch.rand(n, 3, **f64) * 2 - 1
        w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
        rot = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                           2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                           2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], 1).reshape(n, 3, 3)
        scale = 0.1 + 0.3 * torch.rand(n, 3, **f64)
    else:
        d = q[:, :3] / q[:, :3].norm(dim=1, keepdim=True)
        omega, amp = 3 * torch.randn(8, 3, **f64), torch.rand(8, **f64) * 2 - 1
        phase = 2 * math.pi * torch.rand(8, **f64)
        noise = (amp * torch.sin(d @ omega.T + phase)).mean(1)
        pos = (0.8 * (1 + 0.1 * noise))[:, None] * d + 0.01 * torch.randn(n, 3, **f64)
        up = torch.zeros(n, 3, dtype=torch.float64, device=DEV)
        up[:, 0] = (d[:, 1].abs() >= 0.9).double()
        up[:, 1] = 1 - up[:, 0]
        x0 = torch.linalg.cross(up, d)
        x0 = x0 / x0.norm(dim=1, keepdim=True)
        y0 = torch.linalg.cross(d, x0)
        t = 2 * math.pi * torch.rand(n, 1, **f64)
        rot = torch.stack([t.cos() * x0 + t.sin() * y0, -t.sin() * x0 + t.cos() * y0, d], -1)
        scale = _extent(c) * (0.9 + 0.2 * torch.rand(n, 3, **f64))
    pay = torch.rand(n, m, m, m, 4, dtype=torch.float32, device=DEV, generator=gen)
    pay[..., 3] *= 4.0
    if c["empty"] > 0:
        pay[..., 3] *= torch.rand(n, m, m, m, dtype=torch.float32, device=DEV, generator=gen) >= c["empty"]
    if c["bf16"]:
        pay = pay.to(torch.bfloat16)
    return DevicePrims(pos.float().contiguous(), rot.float().contiguous(), scale.float().contiguous(), pay)


def _camera(rng, width, height):
    """Pinhole camera on the sphere of radius 3 looking at the origin, focal length = width."""
    w = rng.normal(size=3)
    w /= np.linalg.norm(w)
    right = np.cross(-w, [0.0, 1.0, 0.0] if abs(w[1]) <= 0.99 else [1.0, 0.0, 0.0])
    right /= np.linalg.norm(right)
    r_cw = np.stack([right, np.cross(-w, right), -w], axis=1)
    k_inv = np.array([[1.0, 0.0, -0.5 * width], [0.0, 1.0, -0.5 * height], [0.0, 0.0, width]]) / width
    return Camera(width, height, (3.0 * w).astype(np.float32), (r_cw @ k_inv).astype(np.float32))


class _Scenes:
    """Resident scenes of one state, released with it."""

    def __init__(self, server, prims):
        self.server, self.ids = server, [server.add_scene(p) for p in prims]

    def __del__(self):
        for i in self.ids:
            self.server.release_scene(i)


def _inputs(case, seed):
    """Everything drawn from the seed, before any handle is made of it."""
    c = case
    gen = torch.Generator(DEV).manual_seed(int(seed))
    rng = np.random.default_rng(int(seed))
    s = {"case": c, "params": MarchParams(1.0 / c["steps"], EPS, fade_alpha=c["fade"], combine=c["combine"])}
    if c["kind"] == "serve":
        s["scenes"] = [_scene(c, gen) for _ in range(4)]
        res = [SERVE_RESOLUTIONS[i % len(SERVE_RESOLUTIONS)] for i in range(c["requests"])]
        s["requests"] = [(int(rng.integers(0, 4)), _camera(rng, w, h)) for w, h in res]
        return s
    s["prims"] = _scene(c, gen)
    s["cams"] = [_camera(rng, c["width"], c["height"]) for _ in range(c["views"])]
    px = c["views"] * c["height"] * c["width"]
    shape = (c["views"], c["height"], c["width"])
    if c["kind"] == "rays":
        s["rays"] = torch.randperm(px, device=DEV, generator=gen)[: c["rays"]].contiguous()
        shape = (c["rays"],)
    s["bg"] = torch.rand(shape + (3,), device=DEV, generator=gen) if c["bg"] else None
    if c["kind"] != "frame":
        s["target"] = torch.rand(shape + (4,), device=DEV, generator=gen)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["ctx"] = _context()
    c = case
    if c["kind"] == "serve":
        s["server"] = Server(s["ctx"], budget_bytes=32 << 30, slots=4)
        torch.cuda.synchronize()     # the scenes are copied on the library's own stream
        s["resident"] = _Scenes(s["server"], s.pop("scenes"))
        s["out"] = [torch.empty((cam.height, cam.width, 4), device=DEV) for _, cam in s["requests"]]
    elif c["kind"] != "frame":
        p = s["prims"]
        s["grads"] = {"payload": torch.zeros(p.payload.shape, device=DEV), "pos": torch.zeros_like(p.pos),
                      "rot": torch.zeros_like(p.rot), "scale": torch.zeros_like(p.scale)}
        if c["bg"]:
            s["grads"]["background"] = torch.zeros_like(s["bg"])
        if _autograd(c):
            for k in ("pos", "rot", "scale", "payload"):
                getattr(p, k).requires_grad_(True)
    return s


def _autograd(c):
    """The steps without a background or a subset on few boxes go through the autograd function."""
    return c["kind"] == "train" and _boxes(c) and not c["bg"]


def _grad_rgba(rgba, target):
    """d mean((rgba - target)^2) / d rgba."""
    return torch.sub(rgba, target).mul_(2.0 / target.numel())


# ----------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------

def run(state):
    s = state
    c, ctx = s["case"], s["ctx"]
    if c["kind"] == "serve":
        srv = s["server"]
        tickets = [srv.submit(s["resident"].ids[i], cam, s["params"], out)
                   for (i, cam), out in zip(s["requests"], s["out"])]
        for t in tickets:
            if srv.wait(t) != 0:
                raise RuntimeError("request not done")
            srv.release(t)
        return s["out"]
    p = s["prims"]
    if _autograd(c):
        leaves = [p.pos, p.rot, p.scale, p.payload]
        rgba = render(ctx, *leaves, s["cams"], s["params"])
        g = torch.autograd.grad(rgba, leaves, _grad_rgba(rgba.detach(), s["target"]))
        return {"rgba": rgba.detach(), **dict(zip(POSE + ("payload",), g))}
    acc = ctx.build_accel(p, s["cams"], s["params"], rays=s.get("rays"))
    back = c["kind"] != "frame"
    rgba, aux = acc.render_fwd(p, want_aux=back, background=s["bg"])
    out = {"rgba": rgba}
    if back:
        g = _grad_rgba(rgba, s["target"])
        for v in s["grads"].values():
            v.zero_()
        out.update(acc.render_bwd(p, aux, g, s["grads"], background=s["bg"], rgba=rgba))
    acc.destroy()
    return out


# ----------------------------------------------------------------------------
# the same in 64 bits
# ----------------------------------------------------------------------------

def exact(case, seed):
    """Each ray's samples are those that the method's binary32 slab test puts inside each box (that test defines them);
    every value and gradient from there on is in 64 bits."""
    c = case
    s = _inputs(c, seed)
    if c["kind"] == "serve":
        return [_Exact(c, s["scenes"][i], [cam], None, None, None).frame(0, cam) for i, cam in s["requests"]]
    e = _Exact(c, s["prims"], s["cams"], s.get("rays"), s["bg"], s.get("target"))
    return e.all()


class _Exact:
    MAX_TESTS, MAX_SAMPLES = 24e6, 6e6     # slab tests and samples held at once

    def __init__(self, c, prims, cams, rays, bg, target):
        self.c, self.cams, self.rays, self.bg, self.target = c, cams, rays, bg, target
        self.back = target is not None
        self.dt = 1.0 / c["steps"]
        self.seq = c["combine"] == "sequential"
        self.p32 = prims
        inv = 1.0 / prims.scale
        self.A32 = prims.rot.transpose(1, 2).contiguous() * inv[:, :, None]     # rows of diag(1/s) R^T
        self.A, self.t = self.A32.double(), prims.pos.double()
        self.R, self.s = prims.rot.double(), prims.scale.double()
        self.vox = prims.payload.detach().reshape(-1, 4)
        m = c["m"]
        x = (-1 + 2 * torch.arange(m, device=DEV, dtype=torch.float64) / (m - 1)).abs()
        w = torch.exp(-c["fade"] * x ** 8.0)
        self.win = (w[:, None, None] * w[None, :, None] * w[None, None, :]).reshape(-1) if c["fade"] > 0 else None
        if self.back:
            self.gp = torch.zeros(self.vox.shape, dtype=torch.float64, device=DEV)
            self.sums = torch.zeros(c["n"], 12, dtype=torch.float64, device=DEV)

    def all(self):
        c = self.c
        px = c["height"] * c["width"]
        shape = (c["views"], c["height"], c["width"]) if self.rays is None else (c["rays"],)
        rgba = torch.zeros(shape + (4,), dtype=torch.float64, device=DEV)
        gbg = torch.zeros(shape + (3,), dtype=torch.float64, device=DEV) if c["bg"] and self.back else None
        for v, cam in enumerate(self.cams):
            if self.rays is None:
                self.frame(v, cam, rgba[v].view(-1, 4), None if gbg is None else gbg[v].view(-1, 3))
            else:
                where = (self.rays // px == v).nonzero().squeeze(1)
                for part in where.split(max(1, int(self.MAX_TESTS // max(1, c["n"])))):
                    self.some(cam, self.rays[part] - v * px, part, rgba, gbg)
        out = {"rgba": rgba}
        if self.back:
            out.update(self.pose(), payload=self.gp.view(self.p32.payload.shape))
            if gbg is not None:
                out["background"] = gbg
        return out

    def frame(self, v, cam, rgba=None, gbg=None):
        """One full view, a few pixel rows at a time."""
        c = self.c
        H, W = cam.height, cam.width
        alone = rgba is None
        if alone:
            rgba = torch.zeros(H * W, 4, dtype=torch.float64, device=DEV)
        per_row = max(1.0, 4.0 * _prim_samples(dict(c, kind="frame", views=1, rays=0, width=W, height=H)) / H)
        rows = int(max(1, min(64, self.MAX_SAMPLES // per_row)))
        bg = None if self.bg is None else self.bg[v].reshape(-1, 3)
        target = None if self.target is None else self.target[v].reshape(-1, 4)
        for y in range(0, H, rows):
            pix = torch.arange(y * W, min(H, y + rows) * W, device=DEV)
            keep = self.near_rows(cam, y, min(H, y + rows))
            step = max(W // 8, int(self.MAX_TESTS // max(1, keep.numel())))
            for part in pix.split(step):
                self.some(cam, part, part, rgba, gbg, keep, bg, target)
        return rgba.view(H, W, 4) if alone else None

    def near_rows(self, cam, y0, y1):
        """Primitives whose bounding sphere may be seen from pixel rows y0 .. y1."""
        P = torch.tensor(cam.pix2dir, dtype=torch.float64, device=DEV)
        rel = self.t - torch.tensor(cam.origin, dtype=torch.float64, device=DEV)
        q = rel @ torch.linalg.inv(P).T
        r = self.s.norm(dim=1) * 1.01
        z, f = q[:, 2], float(cam.width)
        rad = 1.3 * f * r / (z - r).clamp_min(1e-3) + 2
        y = q[:, 1] / z.clamp_min(1e-3)
        return ((z <= 2 * r) | ((y + rad >= y0) & (y - rad <= y1))).nonzero().squeeze(1)

    def some(self, cam, pix, at, rgba, gbg, keep=None, bg=None, target=None):
        """The rays of pixels `pix` of one view; results to rows `at`."""
        c, dt, m = self.c, self.dt, self.c["m"]
        bg = self.bg if bg is None else bg
        target = self.target if target is None else target
        n_rays = pix.numel()
        if keep is None:
            keep = torch.arange(c["n"], device=DEV)
        # binary32 rays, local frames and slab test
        P, o = torch.tensor(cam.pix2dir, device=DEV), torch.tensor(cam.origin, device=DEV)
        u, w = (pix % cam.width).float() + 0.5, (pix // cam.width).float() + 0.5
        e = [(P[i, 0] * u + P[i, 1] * w) + P[i, 2] for i in range(3)]
        nrm = torch.sqrt((e[0] * e[0] + e[1] * e[1]) + e[2] * e[2])
        d = [x / nrm for x in e]
        A = self.A32[keep]
        q = [o[i] - self.p32.pos.detach()[keep, i] for i in range(3)]
        a = [(A[:, i, 0] * q[0] + A[:, i, 1] * q[1]) + A[:, i, 2] * q[2] for i in range(3)]
        lo = torch.zeros(n_rays, keep.numel(), device=DEV)
        hi = torch.full_like(lo, float("inf"))
        miss = torch.zeros_like(lo, dtype=torch.bool)
        for i in range(3):
            b = (A[:, i, 0] * d[0][:, None] + A[:, i, 1] * d[1][:, None]) + A[:, i, 2] * d[2][:, None]
            q0, q1 = (-1 - a[i]) / b, (1 - a[i]) / b
            par = b == 0
            lo = torch.where(par, lo, torch.maximum(lo, torch.minimum(q0, q1)))
            hi = torch.where(par, hi, torch.minimum(hi, torch.maximum(q0, q1)))
            miss |= par & ~((a[i] >= -1) & (a[i] <= 1))
        ray, k = (~miss & (lo <= hi)).nonzero(as_tuple=True)
        j0 = torch.ceil(lo[ray, k].double() / dt).long()     # the step is a power of two: exact
        j1 = torch.floor(hi[ray, k].double() / dt).long()
        del lo, hi, miss
        ok = j0 <= j1
        ray, k, j0, j1 = ray[ok], k[ok], j0[ok], j1[ok]
        a0 = torch.stack(a, 1)[k].double()
        dk = [x[ray] for x in d]
        b0 = torch.stack([(A[k, i, 0] * dk[0] + A[k, i, 1] * dk[1]) + A[k, i, 2] * dk[2] for i in range(3)], 1).double()
        k = keep[k]
        g_out = torch.zeros(n_rays, 4, dtype=torch.float64, device=DEV)
        if ray.numel():
            order = torch.argsort(ray * c["n"] + k)          # by ray, then primitive id
            ray, k, j0, j1, a0, b0 = ray[order], k[order], j0[order], j1[order], a0[order], b0[order]
        # samples of every pair
        cnt = j1 - j0 + 1
        pair = torch.repeat_interleave(torch.arange(cnt.numel(), device=DEV), cnt)
        j = torch.arange(pair.numel(), device=DEV) - (cnt.cumsum(0) - cnt)[pair] + j0[pair]
        tau = j.double() * dt
        h = 0.5 * (m - 1)
        y = (a0[pair] + tau[:, None] * b0[pair]).clamp(-1, 1) * h + h
        cell = y.floor().clamp(max=m - 2)
        f = y - cell
        cell = cell.long()
        base = k[pair] * m ** 3 + (cell[:, 2] * m + cell[:, 1]) * m + cell[:, 0]
        f = f.unbind(1)
        side = [(1 - x, x) for x in f]
        offs = [(i & 1) + m * ((i >> 1) & 1) + m * m * (i >> 2) for i in range(8)]

        def corner(i):
            v = self.vox[base + offs[i]].double()
            if self.win is not None:
                wq = self.win[(base + offs[i]) % m ** 3]
                v = torch.cat([v[:, :3], (v[:, 3] * wq)[:, None]], 1)
                return v, wq
            return v, None

        val = torch.zeros(pair.numel(), 4, dtype=torch.float64, device=DEV)
        for i in range(8):
            val += (side[0][i & 1] * side[1][(i >> 1) & 1] * side[2][i >> 2])[:, None] * corner(i)[0]
        sig, rgb = val[:, 3], val[:, :3]
        # per (ray, sample) sums and the clamped additive accumulation
        jmin = int(j0.min()) if ray.numel() else 0
        J = (int(j1.max()) - jmin + 1) if ray.numel() else 1
        r_of = ray[pair]
        key = r_of * J + (j - jmin)
        S = torch.zeros(n_rays * J, dtype=torch.float64, device=DEV).index_add_(0, key, sig)
        before = (S.view(n_rays, J) * dt).cumsum(1).view(-1) - S * dt    # opacity before each sample
        live = before[key] <= 1 - EPS
        over = live & (before[key] + S[key] * dt > 1)
        wgt = torch.where(live, torch.full_like(sig, dt), torch.zeros_like(sig))
        star = torch.zeros_like(over)
        if self.seq and bool(over.any()):
            # the primitives of a saturating sample one after another by id
            z = over.nonzero().squeeze(1)
            z = z[torch.argsort(key[z], stable=True)]
            step = sig[z] * dt
            cum = step.cumsum(0) - step
            new = torch.ones_like(z, dtype=torch.bool)
            new[1:] = key[z][1:] != key[z][:-1]
            first = torch.where(new, torch.arange(z.numel(), device=DEV), torch.zeros_like(z)).cummax(0).values
            room = 1 - before[key[z]] - (cum - cum[first])
            star[z] = (room >= 0) & (step > room)
            wgt[z] = torch.where(step > 0, torch.minimum(room.clamp_min(0), step) / sig[z].clamp_min(1e-300),
                                 torch.full_like(step, dt))
            wgt[z] = torch.where(room < 0, torch.zeros_like(step), wgt[z])
        elif bool(over.any()):
            wgt = torch.where(over, (1 - before[key]) / S[key].clamp_min(1e-300), wgt)
        acc = torch.zeros(n_rays, 4, dtype=torch.float64, device=DEV)
        acc.index_add_(0, r_of, torch.cat([rgb * (sig * wgt)[:, None], (sig * wgt)[:, None]], 1))
        out = acc.clone()
        if bg is not None:
            out[:, :3] += (1 - acc[:, 3:]) * bg[at].double()
        rgba[at] = out
        if not self.back:
            return
        g_out = (out - target[at].double()) * (2.0 / self.target.numel())
        if gbg is not None:
            gbg[at] = (1 - acc[:, 3:]) * g_out[:, :3]
        # adjoint: dL/dA of unclamped rays, minus the clamping sample's colour of the others
        tdot = g_out[:, 3].clone()
        if bg is not None:
            tdot -= (g_out[:, :3] * bg[at].double()).sum(1)
        g3 = g_out[:, :3][r_of]
        gc = (g3 * rgb).sum(1)
        hit = torch.zeros(n_rays, dtype=torch.bool, device=DEV)
        hit[r_of[over]] = True
        if bool(over.any()):
            share = star.double() if self.seq else torch.where(over, sig / S[key].clamp_min(1e-300), torch.zeros_like(sig))
            mean = torch.zeros(n_rays, dtype=torch.float64, device=DEV).index_add_(0, r_of, share * gc)
            tdot = torch.where(hit, -mean, tdot)
        gsig = wgt * (tdot[r_of] + gc)
        if self.seq:
            gsig = torch.where(star, torch.zeros_like(gsig), gsig)
        adj = torch.cat([g3 * (wgt * sig)[:, None], gsig[:, None]], 1)
        gy = torch.zeros(pair.numel(), 3, dtype=torch.float64, device=DEV)
        for i in range(8):
            v, wq = corner(i)
            sx, sy, sz = side[0][i & 1], side[1][(i >> 1) & 1], side[2][i >> 2]
            dot = (adj * v).sum(1)
            gy[:, 0] += dot * sy * sz * (1 if i & 1 else -1)
            gy[:, 1] += dot * sx * sz * (1 if i & 2 else -1)
            gy[:, 2] += dot * sx * sy * (1 if i & 4 else -1)
            out_v = adj * (sx * sy * sz)[:, None]
            if wq is not None:
                out_v[:, 3] *= wq
            self.gp.index_add_(0, base + offs[i], out_v)
        gy *= h
        pairs = torch.zeros(cnt.numel(), 6, dtype=torch.float64, device=DEV)
        pairs.index_add_(0, pair, torch.cat([gy, gy * tau[:, None]], 1))
        G, H = pairs[:, :3], pairs[:, 3:]
        dd = torch.stack(d, 1).double()[ray]
        M = o.double()[None, :, None] * G[:, None, :] + dd[:, :, None] * H[:, None, :]
        self.sums.index_add_(0, k, torch.cat([G, M.reshape(-1, 9)], 1))

    def pose(self):
        """y = A (o + tau d - t), A = diag(1/s) R^T."""
        G, M = self.sums[:, :3], self.sums[:, 3:].view(-1, 3, 3)
        M = M - self.t[:, :, None] * G[:, None, :]
        return {"pos": -(self.A * G[:, :, None]).sum(1), "rot": M / self.s[:, None, :],
                "scale": -(self.R * M).sum(1) / self.s ** 2}
