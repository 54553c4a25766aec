"""Performance cases of the PackUV-GS splatting path.

A case names one thing that a fitting or viewing program has the framework
do: a fitting step (fetch, projection, bin/sort, compositing, loss, adjoint),
a forward render, the photometric loss, flow masking, UV pruning or the sparse
Adam update.  Scenes are drawn on the GPU from a seed, with the distributions
of the framework's synthetic workloads: positions U([-1, 1]^3), log-scales
N(mu, 0.5), logit-opacities N(0, 1), SH N(0, 0.2), cameras at radius 4 on a
ring or a Fibonacci sphere looking at the origin with a 60 degree field of
view.

``exact`` restates the method in torch FP64 (projection, per-pixel compositing
over per-tile lists, losses; the adjoint by autograd).
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2602_23040_amd import _abi as abi
from paper_2602_23040_amd.pipeline import PackUVRender, Renderer

DEV = "cuda:0"
LAMBDA_SSIM, S_MAX, W_REG = 0.2, 0.05, 1e-4
ADAM = {"lr": 1e-3, "b1": 0.9, "b2": 0.999, "eps": 1e-8}
ADAM_T = 100                # the moments are those of a fit under way


def _case(name, kind, aw, ah, occ, sh, frames, views, w, h, **more):
    """aw x ah atlas, occupied share, SH degree, frames, views per frame, view size."""
    c = {"name": name, "kind": kind, "aw": aw, "ah": ah, "occ": occ, "sh": sh, "frames": frames, "views": views,
         "w": w, "h": h, "ragged": False, "lscale": -5.0, "tiling": "16x16x256", "mode": "eager", "lpo": False,
         "frozen": False, "full": False}
    c.update(more)
    return c


def listed():
    return [
        # a first small fit, driven step by step with the defaults: one 128^2 view of a 64^2 atlas
        _case("step one 128sq view", "step", 64, 64, 1.0, 0, 1, 1, 128, 128, lscale=-4.0),
        # the usual small capture: a ring of eight 512^2 cameras, the step captured in a graph
        _case("step ring of 8", "step", 256, 256, 1.0, 3, 1, 8, 512, 512, mode="graph", tiling="32x8x64"),
        # the renderer inside somebody's own torch loss: odd sizes, a half-empty atlas
        _case("autograd odd sizes", "step", 201, 150, 0.55, 2, 1, 3, 501, 333, mode="autograd", lscale=-4.5),
        # the 360-degree rig: 50 cameras of 1024x768 around a 293k-Gaussian multi-scale atlas
        _case("step 50 views", "step", 896, 512, 0.638, 3, 1, 50, 1024, 768, mode="graph", tiling="16x16x64"),
        # a temporal window: ragged 1080p / 720p cameras per frame, low-precision proxy, gradient freezing
        _case("step window of 4 frames", "step", 1024, 1024, 0.6, 3, 4, 8, 1920, 1080, ragged=True, mode="graph",
              tiling="16x16x128", lpo=True, frozen=True),
        # the largest atlas, ten 1080p cameras
        _case("step 2048sq atlas", "step", 2048, 2048, 0.75, 3, 1, 10, 1920, 1080, mode="graph", tiling="16x16x128",
              lscale=-6.0),
        # the full objective (L1/SSIM blend and both regularisers), driven step by step
        _case("step full objective", "step", 512, 512, 0.8, 3, 1, 16, 800, 600, full=True, tiling="16x16x64"),
        # a viewer: one 1080p image of 293k Gaussians, forward only
        _case("view 1080p", "view", 896, 512, 0.638, 3, 1, 1, 1920, 1080, tiling="16x16x64"),
        # the photometric loss alone, as a program with another renderer state calls it
        _case("photometric loss", "photo", 32, 32, 1.0, 0, 1, 16, 1024, 768, full=True),
        # labels for gradient freezing: every Gaussian against the motion masks of 50 cameras
        _case("flow masking", "flow", 896, 512, 0.638, 3, 1, 50, 1024, 768),
        # UV pruning after a densification of a window of frames
        _case("UV pruning", "prune", 1024, 1024, 0.6, 0, 2, 1, 64, 64),
        # the optimiser's update of the largest atlas
        _case("sparse Adam 2048sq", "adam", 2048, 2048, 0.75, 3, 1, 4, 1920, 1080, lscale=-6.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "step", "view", "view", "photo", "flow", "prune", "adam"])
    while True:
        side = _log(rng, 48, 2048)
        aw, ah = side, max(16, int(side * rng.uniform(0.5, 1.0)))
        occ = round(rng.uniform(0.4, 1.0), 3)
        w = _log(rng, 96, 1920)
        h = max(32, int(w * rng.uniform(0.5, 1.0)))
        frames = rng.choice([1, 1, 1, 2, 3, 4])
        views = 1 if kind == "view" else _log(rng, 1, 50)
        n_gv, px = aw * ah * occ * views * frames, w * h * views * frames
        if n_gv <= 2.5e7 and px <= 3.5e7 and aw * ah * frames <= 4.2e6:
            break
    mode = rng.choice(["eager", "graph", "graph", "autograd"]) if kind == "step" else "eager"
    full = kind == "photo" or (kind == "step" and mode != "autograd" and rng.random() < 0.25)
    return _case("", kind, aw, ah, occ, rng.choice([0, 1, 2, 3, 3, 3]), frames, views, w, h, mode=mode, full=full,
                 ragged=views > 1 and rng.random() < 0.3, frozen=kind == "step" and rng.random() < 0.3, lpo=kind in ("step", "view") and rng.random() < 0.25,
                 lscale=round(-4.0 - math.log2(max(side, 64) / 64) / 2.5 + rng.uniform(-0.2, 0.2), 3),
                 tiling=rng.choice(["16x16x256", "16x16x64", "16x16x128", "32x8x64", "8x32x128"])) | {"name": "drawn"}


# ----------------------------------------------------------------------------- scenes

def _cameras(case):
    cams, n = [], case["views"]
    golden = math.pi * (3.0 - math.sqrt(5.0))
    for f in range(case["frames"]):
        for k in range(n):
            if n > 10:                       # Fibonacci sphere
                z = 1.0 - 2.0 * (k + 0.5) / n
                rho, phi = math.sqrt(1.0 - z * z), k * golden
                eye = 4.0 * np.array([rho * math.cos(phi), rho * math.sin(phi), z])
            else:                            # ring
                a = 2.0 * math.pi * k / n
                eye = 4.0 * np.array([math.cos(a), math.sin(a), 0.0])
            fwd = -eye / np.linalg.norm(eye)
            right = np.cross(fwd, (0.0, 0.0, 1.0))
            right /= np.linalg.norm(right)
            R = np.stack([right, np.cross(fwd, right), fwd])
            w, h = case["w"], case["h"]
            if case["ragged"] and k % 2:
                w, h = max(1, 2 * w // 3), max(1, 2 * h // 3)
            fl = w / (2.0 * math.tan(math.radians(30.0)))
            cams.append(SimpleNamespace(R=R, t=-R @ eye, fx=fl, fy=fl, cx=w / 2.0, cy=h / 2.0, width=w, height=h,
                                        frame=f))
    return cams


def _occupancy(case, seed):
    """Occupied texels, chosen at random; their number depends on the case alone."""
    tex = case["ah"] * case["aw"]
    n = max(1, round(case["occ"] * tex))
    occ = np.zeros(tex, np.uint8)
    occ[np.argpartition(np.random.default_rng([seed, 17]).random(tex, np.float32), n - 1)[:n]] = 1
    return occ.reshape(case["ah"], case["aw"])


def _channels(case):
    return 11 + 3 * (case["sh"] + 1) ** 2


def _atlas(case, gen, occ):
    F, C, H, W = case["frames"], _channels(case), case["ah"], case["aw"]
    a = torch.empty((F, C, H, W), dtype=torch.float32, device=DEV)
    a[:, 0:3].uniform_(-1.0, 1.0, generator=gen)
    a[:, 3:6].normal_(case["lscale"], 0.5, generator=gen)
    a[:, 6:10].normal_(0.0, 1.0, generator=gen)
    a[:, 10].normal_(0.0, 1.0, generator=gen)
    a[:, 11:].normal_(0.0, 0.2, generator=gen)
    return (a * torch.from_numpy(occ).to(DEV)).reshape(-1)


def _gen(seed):
    return torch.Generator(DEV).manual_seed(int(seed))


def _frozen_mask(case, seed):
    rng = np.random.default_rng([seed, 23])
    return (rng.random((case["ah"], case["aw"])) < 0.2).astype(np.uint8) if case["frozen"] else None


def _smooth(cams, gen, channels, cell):
    """Per view, blobs of about `cell` pixels with values around 0.5: flat, the views one after the other."""
    out = []
    for c in cams:
        low = torch.rand((1, channels, c.height // cell + 2, c.width // cell + 2), device=DEV, generator=gen)
        out.append(torch.nn.functional.interpolate(low, (c.height, c.width), mode="bilinear").reshape(-1))
    return torch.cat(out)


def _photo_images(case, gen, cams):
    target = _smooth(cams, gen, 3, 16)
    image = (target + 0.05 * torch.randn(target.shape, device=DEV, generator=gen)).clamp_(0.0, 1.0)
    return image, target


def _flow_masks(gen, cams):
    """uint8 motion masks: blobs over a few per cent of each view."""
    return (_smooth(cams, gen, 1, 40) > 0.85).to(torch.uint8)


def prepare(case, seed):
    gen, occ, cams = _gen(seed), _occupancy(case, seed), _cameras(case)
    s = SimpleNamespace(case=case, graph=None)
    bits = abi.lpo_bits(_channels(case)) if case["lpo"] else None
    r = Renderer(occ, case["frames"], case["sh"], cams, tiling=tuple(int(x) for x in case["tiling"].split("x")),
                 dynamic=_frozen_mask(case, seed), device=DEV, quant_bits=bits)
    s.r, s.atlas = r, _atlas(case, gen, occ)
    kind = case["kind"]
    if kind == "step":
        # the target: another Gaussian set seen by the same cameras
        r.forward(_atlas(case, gen, occ))
        s.target = r.image.clone()
        if case["mode"] == "autograd":
            s.cotangent = torch.randn(r.image.shape, device=DEV, generator=gen) / r.image.numel()
        r.forward(s.atlas)                   # sizes the instance buffers
        s.more = {"lambda_ssim": LAMBDA_SSIM, "reg": {"s_max": S_MAX, "w_scale": W_REG, "w_opacity": W_REG}} \
            if case["full"] else {}
        if case["mode"] == "graph":
            r.check_overflow = False
            main, side = torch.cuda.current_stream(), torch.cuda.Stream()
            side.wait_stream(main)
            with torch.cuda.stream(side):
                r.step(s.atlas, s.target, **s.more)
            main.wait_stream(side)
            torch.cuda.synchronize()
            s.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s.graph):
                r.step(s.atlas, s.target, **s.more)
    elif kind == "view":
        r.forward(s.atlas)
    elif kind == "photo":
        image, s.target = _photo_images(case, gen, cams)
        r.image.copy_(image)
    elif kind == "flow":
        s.masks = _flow_masks(gen, cams)
    elif kind == "adam":
        r.forward(s.atlas)                   # which Gaussians are visible
        _adam_state(r, s.atlas, gen)
    return s


def _adam_state(r, atlas, gen):
    r.dL_datlas.normal_(0.0, 1e-3, generator=gen)
    r.adam_m = torch.empty_like(atlas).normal_(0.0, 3e-4, generator=gen)
    r.adam_v = torch.empty_like(atlas).uniform_(1e-7, 2e-6, generator=gen)
    r.adam_t = torch.full((1,), ADAM_T, dtype=torch.int32, device=DEV)


def run(s):
    r, case = s.r, s.case
    kind = case["kind"]
    if kind == "step":
        if case["mode"] == "autograd":
            atlas = s.atlas.detach().requires_grad_(True)
            img = PackUVRender.apply(atlas, r)
            (img * s.cotangent).sum().backward()
            return {"image": img.detach(), "grad": atlas.grad}
        if s.graph is not None:
            s.graph.replay()
        else:
            r.step(s.atlas, s.target, **s.more)
        return {"loss": r.loss, "image": r.image, "grad": r.dL_datlas}
    if kind == "view":
        return {"image": r.forward(s.atlas)}
    if kind == "photo":
        return {"loss": r.loss_photo(s.target, LAMBDA_SSIM), "dL_dimage": r.dL_dimage}
    if kind == "flow":
        gauss, texel = r.flow_mask(s.atlas, s.masks)
        return {"gauss": gauss, "texel": texel}
    if kind == "prune":
        uv, rank, keep = r.uv_prune(s.atlas, 512, 256, 2)
        return {"uv": uv, "rank": rank, "keep": keep}
    r.adam_step(s.atlas, **ADAM)
    return {"atlas": s.atlas, "m": r.adam_m, "v": r.adam_v}


def work(case):
    """Bytes: the texels (of occupied texels where only those are read), images, masks, gradient and moments, once
    each.  Flops: per (view, Gaussian) 300 for the projection and 600 for its adjoint; per pixel inside the
    3-sigma ellipse (its expected area, at distance 4) 21 for the compositing and 43 for its adjoint."""
    F, C, tex = case["frames"], _channels(case), case["aw"] * case["ah"]
    n = tex * case["occ"]
    px = sum(c.width * c.height for c in _cameras(case))
    n_gv = n * F * case["views"]
    sigma2 = (case["w"] / 1.1547 / 4.0) ** 2 * math.exp(2 * case["lscale"] + 0.5) + 0.3
    pairs = n_gv * math.pi * 9.0 * sigma2 * 0.7
    read = 4 * F * C * n + tex
    kind = case["kind"]
    if kind == "step":
        photo = 3 * px * 392 if case["full"] else 0
        return {"bytes": read + 4 * F * C * tex + 24 * px, "flops": n_gv * 900 + pairs * 64 + photo}
    if kind == "view":
        return {"bytes": read + 12 * px, "flops": n_gv * 300 + pairs * 21}
    if kind == "photo":
        return {"bytes": 36 * px, "flops": 3 * px * 392}
    if kind == "flow":
        return {"bytes": 4 * F * 10 * n + tex + px + F * n + tex, "flops": n_gv * 300}
    if kind == "prune":
        return {"bytes": F * n * (16 + 9) + tex, "flops": F * n * 60}
    return {"bytes": 28 * F * C * n + 5 * F * tex, "flops": 14 * F * C * n}


# ----------------------------------------------------------------------------- the method in 64 bits

def _sh(deg, x, y, z):
    pi = math.pi
    out = [torch.full_like(x, 0.5 * math.sqrt(1 / pi))]
    if deg > 0:
        k = math.sqrt(3 / (4 * pi))
        out += [-k * y, k * z, -k * x]
    if deg > 1:
        k = 0.5 * math.sqrt(15 / pi)
        out += [k * x * y, -k * y * z, 0.25 * math.sqrt(5 / pi) * (3 * z * z - 1), -k * x * z,
                0.5 * k * (x * x - y * y)]
    if deg > 2:
        a, b, k = math.sqrt(35 / (32 * pi)), math.sqrt(21 / (32 * pi)), math.sqrt(105 / (4 * pi))
        out += [-a * y * (3 * x * x - y * y), k * x * y * z, -b * y * (5 * z * z - 1),
                0.25 * math.sqrt(7 / pi) * z * (5 * z * z - 3), -b * x * (5 * z * z - 1),
                0.5 * k * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return torch.stack(out)


def _project(p, cam, deg):
    """Mean [n, 2], conic (a, b, c) and covariance entries, opacity, colour [n, 3], depth and the cull of the
    Gaussians p [C, n] (FP64)."""
    t = {"dtype": torch.float64, "device": p.device}
    R, tr = torch.tensor(np.asarray(cam.R), **t), torch.tensor(np.asarray(cam.t), **t)
    xc, yc, zc = R @ p[0:3] + tr[:, None]
    w, x, y, z = p[6:10] / p[6:10].norm(dim=0)
    Rq = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                      2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                      2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]).reshape(3, 3, -1)
    M = Rq * torch.exp(p[3:6])[None]
    zero = torch.zeros_like(zc)
    J = torch.stack([cam.fx / zc, zero, -cam.fx * xc / zc ** 2, zero, cam.fy / zc,
                     -cam.fy * yc / zc ** 2]).reshape(2, 3, -1)
    T = (J[:, :, None] * (R[:, :, None, None] * M[None]).sum(1)[None]).sum(1)          # J R M: [2, 3, n]
    A, B, Cc = (T[0] ** 2).sum(0) + 0.3, (T[0] * T[1]).sum(0), (T[1] ** 2).sum(0) + 0.3
    det = A * Cc - B * B
    mean = torch.stack([cam.fx * xc / zc + cam.cx, cam.fy * yc / zc + cam.cy], 1)
    d = p[0:3] + (R.T @ tr)[:, None]
    d = d / d.norm(dim=0)
    k = p[11:].reshape((deg + 1) ** 2, 3, -1)
    color = torch.clamp_min(0.5 + (_sh(deg, *d)[:, None] * k).sum(0), 0.0).T
    return mean, torch.stack([Cc, -B, A], 1) / det[:, None], (A, Cc), torch.sigmoid(p[10]), color, zc, \
        (zc > 0.2) & (det > 1e-7)


def _lists(mean, cov, z, ok, w, h, ts=16):
    """(tile, Gaussian) pairs of every ellipse's bounding box, by tile and then front to back."""
    ids = torch.nonzero(ok).reshape(-1)
    ids = ids[torch.sort(z[ids].float(), stable=True).indices]
    m, e = mean[ids], 3.01 * torch.stack([cov[0][ids], cov[1][ids]], 1).sqrt() + 1.0
    nt = torch.tensor([-(-w // ts), -(-h // ts)], device=z.device)
    lo, hi = torch.floor((m - e) / ts).long().clamp_min(0), torch.minimum(torch.floor((m + e) / ts).long(), nt - 1)
    n = (hi - lo + 1).clamp_min(0)
    count = n[:, 0] * n[:, 1]
    who = torch.repeat_interleave(torch.arange(len(ids), device=z.device), count)
    k = torch.arange(len(who), device=z.device) - (torch.cumsum(count, 0) - count)[who]
    tile = (lo[who, 1] + k // n[who, 0]) * nt[0] + lo[who, 0] + k % n[who, 0]
    tile, order = torch.sort(tile, stable=True)
    return tile, ids[who[order]], int(nt[0]), int(nt[0] * nt[1])


def _chunks(tile, n_tiles, most):
    """Groups of tiles with lists of similar length: (tiles, longest list)."""
    length = torch.bincount(tile, minlength=n_tiles)
    order = torch.argsort(length, descending=True)
    sizes, at = length[order].tolist(), 0
    while at < n_tiles:
        L = max(sizes[at], 1)
        step = max(1, most // L)
        yield order[at:at + step], L
        at += step


def _composite(rows, L, start, length, who, splat, w, h, tx, ts=16):
    """Colours [B, 256, 3], pixel indices and which of them lie inside the view, for a group of tiles."""
    mean, conic, opac, color = splat
    px = torch.arange(ts, device=rows.device)
    X = ((rows % tx) * ts)[:, None] + px.repeat(ts)[None]
    Y = ((rows // tx) * ts)[:, None] + px.repeat_interleave(ts)[None]
    j = torch.arange(L, device=rows.device)
    have = j[None] < length[rows][:, None]
    g = who[(start[rows][:, None] + j[None]).clamp_max(max(len(who) - 1, 0))] if len(who) else \
        torch.zeros((len(rows), L), dtype=torch.long, device=rows.device)
    dx = (X + 0.5)[:, :, None] - mean[g, 0][:, None]
    dy = (Y + 0.5)[:, :, None] - mean[g, 1][:, None]
    a, b, c = (conic[g, i][:, None] for i in range(3))
    q = a * dx * dx + 2 * b * dx * dy + c * dy * dy
    alpha = torch.clamp_max(opac[g][:, None] * torch.exp(-0.5 * q), 0.99)
    take = have[:, None] & (q <= 9) & (alpha >= 1 / 255)
    keep = torch.cumprod(torch.where(take, 1 - alpha, 1.0), 2)
    take = take & (keep.detach() >= 1e-4)
    alpha = torch.where(take, alpha, 0.0)
    T = torch.cumprod(1 - alpha, 2)
    T = torch.cat([torch.ones_like(T[:, :, :1]), T[:, :, :-1]], 2)
    return torch.matmul(T * alpha, color[g].contiguous()), Y * w + X, (X < w) & (Y < h)


def _ssim(x, y):
    """Mean of the SSIM map over the planes x, y [n, H, W] (11 x 11 Gaussian window, sigma 1.5, zero padding)."""
    k = torch.arange(11, dtype=torch.float64, device=x.device) - 5
    k = torch.exp(-k * k / (2 * 1.5 ** 2))
    k = k / k.sum()

    def blur(v):
        H, W = v.shape[1:]
        v = torch.nn.functional.pad(v, (0, 0, 5, 5))
        v = sum(k[i] * v[:, i:i + H] for i in range(11))
        v = torch.nn.functional.pad(v, (5, 5))
        return sum(k[i] * v[:, :, i:i + W] for i in range(11))
    mx, my = blur(x), blur(y)
    sx, sy, sxy = blur(x * x) - mx * mx, blur(y * y) - my * my, blur(x * y) - mx * my
    C1, C2 = 0.01 ** 2, 0.03 ** 2
    return ((2 * mx * my + C1) * (2 * sxy + C2)) / ((mx * mx + my * my + C1) * (sx + sy + C2))


def _loss(case, image, target, cams):
    """The photometric loss of flat images (FP64) and its image gradient."""
    image = image.detach().requires_grad_(True)
    lam, n, at, parts = LAMBDA_SSIM if case["full"] else 0.0, image.numel(), 0, []
    for c in cams:
        size = 3 * c.width * c.height
        x, y = (v[at:at + size].reshape(3, c.height, c.width) for v in (image, target))
        part = (1 - lam) * (x - y).abs().sum()
        if lam:
            part = part + lam * (x.numel() - _ssim(x, y).sum())
        (part / n).backward()
        parts.append(part.detach() / n)
        at += size
    return sum(parts), image.grad


def _render(case, params, cams, frames_n, cotangent=None):
    """The flat image of every view, and with a cotangent the gradient of the parameters [F][C][N]."""
    deg, out, at = case["sh"], [], 0
    leaf = params.detach().requires_grad_(cotangent is not None)
    for cam in cams:
        with torch.set_grad_enabled(cotangent is not None):
            mean, conic, cov, opac, color, z, ok = _project(leaf[cam.frame], cam, deg)
        w, h = cam.width, cam.height
        with torch.no_grad():
            tile, who, tx, n_tiles = _lists(mean, cov, z, ok, w, h)
            length = torch.bincount(tile, minlength=n_tiles)
            start = torch.cumsum(length, 0) - length
        splat = [v.detach().requires_grad_(cotangent is not None) for v in (mean, conic, opac, color)]
        img = torch.zeros((3, w * h), dtype=torch.float64, device=params.device)
        for rows, L in _chunks(tile, n_tiles, 1 << 16):
            with torch.set_grad_enabled(cotangent is not None):
                col, pix, inside = _composite(rows, L, start, length, who, splat, w, h, tx)
            img[:, pix[inside]] = col.detach()[inside].T
            if cotangent is not None and col.requires_grad:
                g = cotangent[at:at + 3 * w * h].reshape(3, w * h)
                G = torch.zeros_like(col)
                G[inside] = g[:, pix[inside]].T
                col.backward(G)
        if cotangent is not None and all(v.grad is not None for v in splat):
            torch.autograd.backward([mean, conic, opac, color],
                                    [v.grad * ok.reshape(-1, *[1] * (v.dim() - 1)) for v in splat])
        out.append(img.reshape(-1))
        at += 3 * w * h
    return torch.cat(out), leaf.grad


def exact(case, seed):
    kind = case["kind"]
    if kind in ("flow", "prune"):
        return None
    gen, occ, cams = _gen(seed), _occupancy(case, seed), _cameras(case)
    if kind == "photo":
        _atlas(case, gen, occ)               # drawn before the images
        image, target = (v.double() for v in _photo_images(case, gen, cams))
        loss, g = _loss(case, image, target, cams)
        return {"loss": loss.reshape(1), "dL_dimage": g}
    n, px = int(occ.sum()), sum(c.width * c.height for c in cams)
    F, C, H, W = case["frames"], _channels(case), case["ah"], case["aw"]
    if kind == "adam":
        return None if F * C * H * W > 1.3e8 else _exact_adam(case, seed, gen, occ, cams)
    # the per-tile lists are walked for every pixel in 64 bits: small scenes only
    if case["lpo"] or n * len(cams) > 1.5e6 or px > 4e6:
        return None
    texel = torch.from_numpy(np.flatnonzero(occ.reshape(-1))).to(DEV)
    planes = _atlas(case, gen, occ)
    params = planes.reshape(F, C, H * W)[:, :, texel].double()
    if kind == "view":
        return {"image": _render(case, params, cams, n)[0]}
    other = _atlas(case, gen, occ)
    image = _render(case, params, cams, n)[0]
    if case["mode"] == "autograd":
        G = (torch.randn(image.shape, device=DEV, generator=gen) / image.numel()).double()
    else:
        # the target is the framework's own rendering in 32 bits of the other set
        r = Renderer(occ, F, case["sh"], cams, tiling=(16, 16, 256), device=DEV)
        target = r.forward(other).clone().double()
        r.close()
        loss, G = _loss(case, image, target, cams)
    grad = _render(case, params, cams, n, G)[1]
    if case["frozen"]:
        grad = grad * torch.from_numpy(_frozen_mask(case, seed).reshape(-1)).to(DEV)[texel]
    if case["full"]:
        leaf = params.detach().requires_grad_(True)
        s, o = torch.exp(leaf[:, 3:6]).amax(1), torch.sigmoid(leaf[:, 10])
        (W_REG * torch.clamp_min(s - S_MAX, 0).square().mean() + W_REG * (o * (1 - o)).mean()).backward()
        grad = grad + leaf.grad
    full = torch.zeros((F, C, H * W), dtype=torch.float64, device=DEV)
    full[:, :, texel] = grad
    if case["mode"] == "autograd":
        return {"image": image, "grad": full.reshape(-1)}
    return {"loss": loss.reshape(1), "image": image, "grad": full.reshape(-1)}


def _exact_adam(case, seed, gen, occ, cams):
    r = Renderer(occ, case["frames"], case["sh"], cams, device=DEV)
    atlas = _atlas(case, gen, occ)
    r.forward(atlas)                         # the visible set only
    _adam_state(r, atlas, gen)
    F, C, n = case["frames"], _channels(case), int(occ.sum())
    seen = torch.zeros((F, 1, occ.size), dtype=torch.bool, device=DEV)
    texel = torch.from_numpy(np.flatnonzero(occ.reshape(-1))).to(DEV)
    seen[:, 0, texel] = r.visible[:F * n].reshape(F, n) > 0
    p, g, m0, v0 = (x.double().reshape(F, C, -1) for x in (atlas, r.dL_datlas, r.adam_m, r.adam_v))
    b1, b2, t = ADAM["b1"], ADAM["b2"], ADAM_T + 1
    m, v = b1 * m0 + (1 - b1) * g, b2 * v0 + (1 - b2) * g * g
    new = p - ADAM["lr"] * (m / (1 - b1 ** t)) / ((v / (1 - b2 ** t)).sqrt() + ADAM["eps"])
    r.close()
    return {"atlas": torch.where(seen, new, p).reshape(-1), "m": torch.where(seen, m, m0).reshape(-1),
            "v": torch.where(seen, v, v0).reshape(-1)}
