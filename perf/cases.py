"""Performance cases: the work that programs built on this framework have it do.

A case is a plain dict.  ``kind`` says which public entry points it goes through:

  train     one training step: the sites have moved a little (as after an
            optimiser update), ``update_scene``, a differentiable render of
            all views (``walk`` 0: rasteriser, 1: ray walk; ``recompute`` 1:
            no records kept between forward and backward), the squared error
            to the target images, backward.  ``full`` 1 adds the whole
            objective: normal, sparsity and connectivity losses and the
            per-cell statistics that densification and pruning average.
  render    forward images of a resident scene by the rasteriser, as a viewer
            or a serving batch asks for them
  walk      forward images by the ray walk
  adapt     densification and pruning between training steps: both moving
            averages, the new cell set, and the build of its scene

Scenes are the generators' distributions (``uniform``: sites uniform in a
cube; otherwise 80% on 64 flattened Gaussians and 20% in a shell around them)
with the attribute distributions of the package's workloads, drawn on the GPU.
``views`` pinhole cameras of ``width`` x ``height`` look at the origin;
``fisheye`` 1 makes every camera a 180-degree equidistant fisheye, 2 every
second one; ``shrink`` 1 halves the size from each view to the next (a batch
of requests of mixed sizes).
"""
from __future__ import annotations

import math
import types

import numpy as np
import torch

import paper_2604_24994_amd as pf

SIGMA_SCALE, TAU = 10.0, 20.0
K, M = 8, 8
FIELDS = ("p", "power", "radius", "normal", "occ_logit", "rgb", "tex")
LAMBDA_NORMAL, LAMBDA_SPARSE, LAMBDA_CONNECT = 1e-3, 1e-4, 1e-3

DEFAULTS = {"uniform": 0, "views": 1, "width": 0, "height": 0, "fisheye": 0, "shrink": 0, "walk": 0, "recompute": 0,
            "full": 0}


def listed():
    return [
        # the smallest step: unit tests, toy scenes, the first steps from a sparse initialisation
        {"name": "train 1k", "kind": "train", "cells": 1024, "uniform": 1, "width": 128, "height": 128},
        # early training with every loss term and the statistics, odd image sizes
        {"name": "train full 16k", "kind": "train", "cells": 16384, "views": 2, "width": 401, "height": 267, "full": 1},
        # one ordinary training iteration: one full frame of a medium scene
        {"name": "train 262k", "kind": "train", "cells": 262144, "width": 1280, "height": 720},
        # the large training step: a batch of eight views at full size
        {"name": "train 1m", "kind": "train", "cells": 1048576, "views": 8, "width": 1600, "height": 1066},
        # training with bounded memory at the 500K cells of an indoor scene, ragged sizes
        {"name": "train recompute 500k", "kind": "train", "cells": 500000, "views": 2, "width": 1237, "height": 822,
         "recompute": 1},
        # training through the ray walk
        {"name": "train walk 100k", "kind": "train", "cells": 100003, "width": 640, "height": 360, "walk": 1},
        # a thumbnail of a small scene: latency
        {"name": "render 1k", "kind": "render", "cells": 1024, "uniform": 1, "width": 128, "height": 128},
        # the smallest serving request on a large resident scene
        {"name": "render small 1m", "kind": "render", "cells": 1048576, "width": 256, "height": 256},
        # a serving batch of mixed sizes and camera models
        {"name": "render batch 1m", "kind": "render", "cells": 1048576, "views": 4, "width": 1920, "height": 1080,
         "fisheye": 2, "shrink": 1},
        # a small interactive fisheye view by the ray walk
        {"name": "walk fisheye 16k", "kind": "walk", "cells": 16384, "width": 300, "height": 300, "fisheye": 1},
        # a full frame by the ray walk of a large scene
        {"name": "walk 1m", "kind": "walk", "cells": 1048576, "width": 1280, "height": 720},
        # the cell set changes: statistics, prune, draw, and a build from scratch
        {"name": "adapt 300k", "kind": "adapt", "cells": 300000},
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("train", "train", "train", "render", "render", "walk", "adapt"))
    c = {"kind": kind, "cells": log(1000, 1048576)}
    if c["cells"] < 8000:
        c["uniform"] = rng.randrange(2)
    if kind == "adapt":
        return {"kind": kind, "cells": log(4000, 524288)}
    c["width"], c["height"] = log(100, 1920), log(100, 1080)
    c["views"] = rng.choice((1, 1, 2, 3, 5))
    c["fisheye"] = rng.choice((0, 0, 0, 1, 2))
    if kind == "train":
        c["full"] = rng.choice((0, 0, 1))
        c["recompute"] = rng.choice((0, 0, 1))
        c["walk"] = rng.choice((0, 0, 0, 1))
    elif kind == "render":
        c["shrink"] = rng.randrange(2)
    if kind == "walk" or c.get("walk"):
        c["views"] = 1
    return c


def _full(case):
    return {**DEFAULTS, **case}


# --------------------------------------------------------------------------
# inputs


def _params(c, seed):
    """Cell parameters on the GPU, from the seed alone."""
    n = c["cells"]
    g = torch.Generator(device="cuda").manual_seed(seed)

    def rand(*shape, lo=0.0, hi=1.0):
        return torch.rand(*shape, device="cuda", generator=g) * (hi - lo) + lo

    def randn(*shape):
        return torch.randn(*shape, device="cuda", generator=g)

    if c["uniform"]:
        p = rand(n, 3, lo=-1.0, hi=1.0)
    else:
        ns, k = int(round(0.8 * n)), 64
        comp = torch.randint(0, k, (ns,), device="cuda", generator=g)
        sig = torch.cat([rand(k, 2, lo=0.1, hi=0.3), rand(k, 1, lo=0.01, hi=0.05)], 1)
        q, _ = torch.linalg.qr(randn(k, 3, 3).cpu())
        q = q.cuda()
        surf = rand(k, 3, lo=-1.0, hi=1.0)[comp] + (q[comp] * (randn(ns, 3) * sig[comp])[:, None, :]).sum(-1)
        u = torch.nn.functional.normalize(randn(n - ns, 3), dim=1)
        p = torch.cat([surf, u * rand(n - ns, 1, lo=27.0, hi=216.0).pow(1.0 / 3.0)])
    s = rand(n, lo=0.02, hi=0.1)
    return {"p": p.contiguous(), "power": s * s, "radius": 1.5 * s,
            "normal": torch.nn.functional.normalize(randn(n, 3), dim=1), "occ_logit": randn(n), "rgb": rand(n, 3),
            "tex": randn(n, K, 3 + 6 * M).mul_(0.1)}


def _look_at(eye):
    f = -eye / np.linalg.norm(eye)
    up = np.array([0.0, 0.0, 1.0]) if abs(f[2]) < 0.999 else np.array([0.0, 1.0, 0.0])
    right = np.cross(f, up)
    right /= np.linalg.norm(right)
    return np.stack([right, np.cross(f, right), f, eye], axis=1).astype(np.float32)


def _cameras(c, seed):
    rng = np.random.default_rng(seed)
    cams = []
    for v in range(c["views"]):
        e = rng.normal(size=3)
        e *= (3.0 if c["uniform"] else 4.0) / np.linalg.norm(e)
        w, h = c["width"], c["height"]
        if c["shrink"]:
            w, h = max(16, w >> v), max(16, h >> v)
        cam = types.SimpleNamespace(model=0, width=w, height=h, c2w=_look_at(e), fx=0.0, fy=0.0, cx=w / 2.0,
                                    cy=h / 2.0, f_fish=0.0, theta_max=0.0)
        if c["fisheye"] == 1 or (c["fisheye"] == 2 and v % 2 == 1):
            cam.model = 1
            cam.theta_max = float(np.float32(math.pi / 2))
            cam.f_fish = float(np.float32(min(w, h) / 2.0 / (math.pi / 2)))
        else:
            cam.fx = cam.fy = float(np.float32(h / 2.0 / math.tan(math.radians(30.0))))
        cams.append(cam)
    return cams


def _rays(cams):
    return sum(c.width * c.height for c in cams)


def _train_inputs(c, seed):
    params, cams = _params(c, seed), _cameras(c, seed)
    g = torch.Generator(device="cuda").manual_seed(seed + 1)
    move = torch.randn(c["cells"], 3, device="cuda", generator=g) * 1e-4
    target = torch.rand(_rays(cams), 3, device="cuda", generator=g)
    error = torch.rand(_rays(cams), device="cuda", generator=g)
    return params, cams, move, target, error


def _adapt_inputs(c, seed):
    n = c["cells"]
    params = _params(c, seed)
    g = torch.Generator(device="cuda").manual_seed(seed + 2)
    nn = max(1, n // 100)
    # the contributions are spread evenly, in random order: 5% of the cells lie below the threshold
    spread = (torch.randperm(n, device="cuda", generator=g).float() + 0.33) / n
    return params, {"error": torch.rand(n, device="cuda", generator=g),
                    "contribution": spread,
                    "ema_error": torch.rand(n, device="cuda", generator=g),
                    "ema_contribution": spread.clone(),
                    "u": torch.rand(nn, device="cuda", generator=g),
                    "delta": torch.randn(nn, 3, device="cuda", generator=g)}


BETA, PRUNE_BELOW, SPREAD = 0.9, 0.05, 0.5
# the domain box holds every camera, so that the walk can start there
BOX = ((-6.5,) * 3, (6.5,) * 3)
FACES_PER_CELL = 24   # no scene has more on average


def prepare(case, seed):
    c = _full(case)
    if c["kind"] == "adapt":
        params, stats = _adapt_inputs(c, seed)
        return {"case": c, "params": params, "stats": stats}
    if c["kind"] == "train":
        params, cams, move, target, error = _train_inputs(c, seed)
        for v in params.values():
            v.requires_grad_(True)
        scene = pf.build_scene(params, sigma_scale=SIGMA_SCALE, tau=TAU, box=BOX)
        return {"case": c, "params": params, "cams": cams, "move": move, "target": target, "error": error,
                "scene": scene, "sign": 1.0}
    params, cams = _params(c, seed), _cameras(c, seed)
    return {"case": c, "cams": cams, "scene": pf.build_scene(params, sigma_scale=SIGMA_SCALE, tau=TAU, box=BOX)}


# --------------------------------------------------------------------------
# one pass


def run(state):
    kind = state["case"]["kind"]
    if kind == "train":
        return _train_step(state)
    if kind == "render":
        return pf.render_raster(state["scene"], state["cams"])
    if kind == "walk":
        return pf.render_trace(state["scene"], state["cams"])
    return _adapt(state)


def _train_step(state):
    c, params, scene, cams = state["case"], state["params"], state["scene"], state["cams"]
    with torch.no_grad():   # the sites move to and fro between steps
        params["p"].add_(state["move"], alpha=state["sign"])
    state["sign"] = -state["sign"]
    for v in params.values():
        v.grad = None
    pf.update_scene(scene, params)
    stats = {"pixel_error": state["error"]} if c["full"] else None
    render = pf.render_trace_diff if c["walk"] else pf.render_raster_diff
    imgs = render(scene, cams, state_mode=pf.RECOMPUTE if c["recompute"] else pf.STORE,
                  lambda_normal=LAMBDA_NORMAL if c["full"] else 0.0, stats=stats)
    rgba = torch.cat([im.reshape(-1, 4) for im in imgs])
    loss = ((rgba[:, :3] - state["target"]) ** 2).mean()
    if c["full"]:
        loss = loss + LAMBDA_SPARSE * rgba[:, 3].mean()
    loss.backward()
    out = {"images": [im.detach() for im in imgs]}
    grads = {f: params[f].grad for f in FIELDS}
    total = loss.detach()
    if c["full"]:
        connect = pf.connect_loss(scene, LAMBDA_CONNECT, grads)
        total = total + (LAMBDA_NORMAL * stats["normal_loss"] + connect).float()[0]
        out["contribution"], out["error"] = stats["contribution"], stats["error"]
    out["loss"], out["grads"] = total, grads
    return out


def _adapt(state):
    s = state["stats"]
    ema_e = pf.ema_update(s["ema_error"].clone(), s["error"], BETA)
    ema_c = pf.ema_update(s["ema_contribution"].clone(), s["contribution"], BETA)
    cells, err, con, parent = pf.densify_prune(state["params"], ema_e, ema_c, s["u"], s["delta"], PRUNE_BELOW, SPREAD)
    scene = pf.build_scene(cells, sigma_scale=SIGMA_SCALE, tau=TAU, box=BOX)
    row, found = scene.adjacency()
    # neighbour lists in a buffer of fixed size (the number of faces depends on the cells)
    col = torch.full((FACES_PER_CELL * (row.numel() - 1),), -100, dtype=found.dtype, device=found.device)
    col[:found.numel()] = found
    return {"cells": cells, "error": err, "contribution": con, "parent": parent, "row": row, "col": col}


# --------------------------------------------------------------------------
# the work of a pass

# contributions per ray of the scenes (more cells, longer chains) and the
# operations of one contribution (forward, and forward with backward)
FLOPS_FWD, FLOPS_STEP = 1700, 6800


def work(case):
    c = _full(case)
    n = c["cells"]
    cell = 4 * (3 + 1 + 1 + 3 + 1 + 3 + K * (3 + 6 * M))   # parameters of one cell
    if c["kind"] == "adapt":
        return {"bytes": 2 * cell * n + 16 * n + 2 * 64 * n, "flops": 5000.0 * n}
    rays = 0
    for v in range(c["views"]):
        w, h = c["width"], c["height"]
        if c["shrink"]:
            w, h = max(16, w >> v), max(16, h >> v)
        rays += w * h
    depth = 3.0 if c["uniform"] else min(23.0, 1.2 * n ** 0.21)
    if c["kind"] == "train":
        # parameters and targets in, images and gradients out
        return {"bytes": 2 * cell * n + 44 * rays, "flops": rays * depth * FLOPS_STEP + 5000.0 * n}
    seen = min(n, rays)   # cells whose parameters an image can need
    return {"bytes": 16 * rays + cell * seen * 0.3 + 20 * n, "flops": rays * depth * FLOPS_FWD}


# --------------------------------------------------------------------------
# the same outputs in 64 bits

D = torch.float64


def exact(case, seed):
    c = _full(case)
    if c["kind"] == "adapt":
        return _exact_adapt(c, seed)
    cams = _cameras(c, seed)
    if c["cells"] * _rays(cams) > 4.5e9:
        return None   # every step of a ray looks at every cell
    if c["kind"] == "train":
        return _exact_train(c, seed)
    P = {k: v.to(D) for k, v in _params(c, seed).items()}
    with torch.no_grad():
        return [_exact_view(P, cam).reshape(cam.height, cam.width, 4) for cam in cams]


def _exact_adapt(c, seed):
    params, s = _adapt_inputs(c, seed)

    def ema(a, b):   # the averages are float32 values, the draws use them as such
        return (BETA_32 * a.to(D) + (1.0 - BETA_32) * b.to(D)).float()

    e, k = ema(s["ema_error"], s["error"]), ema(s["ema_contribution"], s["contribution"])
    kept = torch.nonzero(k >= float(np.float32(PRUNE_BELOW))).flatten()
    cdf = torch.cumsum(e[kept].to(D), 0)
    at = torch.searchsorted(cdf, s["u"].to(D) * cdf[-1], right=True).clamp_(max=kept.numel() - 1)
    src = torch.cat([kept, kept[at]])
    cells = {f: params[f][src].to(D) for f in FIELDS}
    nk = kept.numel()
    cells["p"][nk:] += SPREAD * params["radius"][kept[at]].to(D)[:, None] * s["delta"].to(D)
    return {"cells": cells, "error": e[src].to(D), "contribution": k[src].to(D), "parent": None, "row": None,
            "col": None}


BETA_32 = float(np.float32(BETA))


def _directions(cam):
    u = torch.arange(cam.width, device="cuda", dtype=D) + 0.5 - float(np.float32(cam.cx))
    v = torch.arange(cam.height, device="cuda", dtype=D) + 0.5 - float(np.float32(cam.cy))
    v, u = torch.meshgrid(v, u, indexing="ij")
    if cam.model == 0:
        d = torch.stack([u / cam.fx, v / cam.fy, torch.ones_like(u)], -1)
        valid = torch.ones_like(u, dtype=torch.bool)
    else:
        rho = (u * u + v * v).sqrt()
        th = rho / cam.f_fish
        valid = th <= cam.theta_max
        sc = torch.where(rho > 0, th.sin() / rho.clamp(min=1e-300), torch.zeros_like(rho))
        d = torch.stack([sc * u, sc * v, th.cos()], -1)
    m = torch.as_tensor(cam.c2w, device="cuda", dtype=D)
    d = (d.reshape(-1, 3)[:, None, :] * m[:, :3][None]).sum(-1)
    return m[:, 3], d / d.norm(dim=1, keepdim=True), valid.reshape(-1)


def _walk_chunk(P, o, d):
    """Cells along the rays o + t d: (ray, cell, previous cell or -1, next cell or -1).
    Along a ray the power distances are lines in t (less the common t^2), so the
    cells met are the lines of their lower envelope, found by stepping from
    crossing to crossing."""
    oc = o[None] - P["p"]
    key = (oc * oc).sum(1) - P["power"]
    slope = d @ oc.T
    nr = d.shape[0]
    ray = torch.arange(nr, device="cuda")
    cell = torch.full((nr,), int(key.argmin()), device="cuda")
    prev = torch.full((nr,), -1, device="cuda")
    out = []
    inf = torch.tensor(math.inf, device="cuda", dtype=D)
    while ray.numel():
        b = slope[ray, cell]
        den = 2.0 * (b[:, None] - slope[ray])
        t = torch.where(den > 0, (key[None] - key[cell][:, None]) / den, inf)
        te, nxt = t.min(1)
        more = torch.isfinite(te)
        out.append((ray, cell, prev, torch.where(more, nxt, torch.full_like(nxt, -1))))
        ray, prev, cell = ray[more], cell[more], nxt[more]
    return [torch.cat(x) for x in zip(*out)]


def _onb(n):
    sign = torch.copysign(torch.ones_like(n[:, 2]), n[:, 2])
    a = -1.0 / (sign + n[:, 2])
    b = n[:, 0] * n[:, 1] * a
    return (torch.stack([1.0 + sign * n[:, 0] ** 2 * a, sign * b, -sign * n[:, 0]], 1),
            torch.stack([b, sign + n[:, 1] ** 2 * a, -n[:, 1]], 1))


def _dot(a, b):
    return (a * b).sum(-1)


def _blend(u, s):
    return torch.softmax(-TAU * (u[:, None] - s).norm(dim=-1), dim=1)


def _crossing(P, o, d, i, j):
    """Ray parameter where the power distances of cells i and j are equal."""
    oi, oj = o[None] - P["p"][i], o[None] - P["p"][j]
    return (_dot(oj, oj) - P["power"][j] - _dot(oi, oi) + P["power"][i]) / (2.0 * _dot(d, oi - oj))


def _shade(P, o, d, i, prev, nxt):
    """Opacity, colour and facing term of the pieces of cells i on the rays d."""
    p, r = P["p"][i], P["radius"][i]
    oc = o[None] - p
    beta = _dot(oc, d)
    sq = (r * r - _dot(oc - beta[:, None] * d, oc - beta[:, None] * d)).clamp(min=1e-300).sqrt()
    lo, hi = (-beta - sq).clamp(min=0.0), -beta + sq
    lo = torch.where(prev >= 0, torch.maximum(lo, _crossing(P, o, d, i, torch.where(prev >= 0, prev, i - 1))), lo)
    hi = torch.where(nxt >= 0, torch.minimum(hi, _crossing(P, o, d, i, torch.where(nxt >= 0, nxt, i - 1))), hi)
    n = P["normal"][i]
    n = n / n.norm(dim=1, keepdim=True)
    t1, t2 = _onb(n)
    tex = P["tex"][i]
    s, disp = tex[..., 0:2], tex[..., 2]
    axes = tex[..., 3:3 + 3 * M].reshape(-1, K, M, 3)
    cols = tex[..., 3 + 3 * M:].reshape(-1, K, M, 3)
    den = _dot(d, n)
    at = -_dot(oc, n) / den
    x = oc + at[:, None] * d
    delta = (_blend(torch.stack([_dot(x, t1), _dot(x, t2)], 1), s) * disp).sum(1)
    tx = at + delta / den
    x = oc + tx[:, None] * d
    w = _blend(torch.stack([_dot(x, t1), _dot(x, t2)], 1), s)
    lo = torch.where(den < 0, torch.maximum(lo, tx), lo)
    hi = torch.where(den > 0, torch.minimum(hi, tx), hi)
    sigma = SIGMA_SCALE * torch.nn.functional.softplus(P["occ_logit"][i])
    alpha = -torch.expm1(-sigma * (hi - lo).clamp(min=0.0))
    v = torch.softmax((axes * d[:, None, None, :]).sum(-1), dim=-1)
    colour = P["rgb"][i] + (w[..., None] * (v[..., None] * cols).sum(2)).sum(1)
    return alpha, colour, _dot(n, d).clamp(min=0.0) ** 2


def _view_chunks(P, cam):
    """Per block of rays: their indices, origin and directions, and the pieces
    with a non-empty dense part: ray within the block, place on the ray, cell,
    previous and next cell."""
    o, dirs, valid = _directions(cam)
    N = P["p"].shape[0]
    at = torch.nonzero(valid).flatten()
    step = max(1, min(1 << 15, int(2.5e9) // N))
    Q = {k: v.detach() for k, v in P.items()}
    for a in range(0, at.numel(), step):
        idx = at[a:a + step]
        d = dirs[idx]
        with torch.no_grad():
            ray, cell, prev, nxt = _walk_chunk(Q, o, d)
            oc = o[None] - Q["p"][cell]
            q = oc - _dot(oc, d[ray])[:, None] * d[ray]
            hit = torch.nonzero(_dot(q, q) < Q["radius"][cell] ** 2).flatten()
            order = hit[torch.sort(ray[hit], stable=True).indices]
            ray, cell, prev, nxt = ray[order], cell[order], prev[order], nxt[order]
            alpha = torch.cat([_shade(Q, o, d[ray[k:k + 200000]], cell[k:k + 200000], prev[k:k + 200000],
                                      nxt[k:k + 200000])[0] for k in range(0, ray.numel(), 200000)] or [oc.new_zeros(0)])
            on = alpha > 0
            ray, cell, prev, nxt = ray[on], cell[on], prev[on], nxt[on]
            count = torch.bincount(ray, minlength=idx.numel())
            place = torch.arange(ray.numel(), device="cuda") - (torch.cumsum(count, 0) - count)[ray]
        yield idx, o, d, ray, place, cell, prev, nxt


def _exact_view(P, cam, objective=None):
    """The image of one view [pixels, 4].  ``objective(idx, rgba, T a per piece,
    facing per piece, cell per piece)`` is differentiated block by block."""
    img = torch.zeros(cam.width * cam.height, 4, device="cuda", dtype=D)
    for idx, o, d, ray, place, cell, prev, nxt in _view_chunks(P, cam):
        if not ray.numel():
            if objective is not None:
                objective(idx, img[idx], None, None, None)
            continue
        # blocks of whole rays, of about 100,000 pieces
        start = torch.searchsorted(ray, torch.arange(idx.numel() + 1, device="cuda"))
        lim, r0 = start.cpu().numpy(), 0
        while r0 < idx.numel():
            r1 = max(r0 + 1, min(idx.numel(), int(np.searchsorted(lim, lim[r0] + 100000, side="right")) - 1))
            k = slice(int(lim[r0]), int(lim[r1]))
            r, pl = ray[k] - r0, place[k]
            alpha, colour, facing = _shade(P, o, d[ray[k]], cell[k], prev[k], nxt[k])
            width = int(pl.max()) + 1 if pl.numel() else 1
            a = torch.zeros(r1 - r0, width, device="cuda", dtype=D).index_put((r, pl), alpha)
            T = torch.cumprod(torch.cat([torch.ones_like(a[:, :1]), 1.0 - a], 1), 1)
            ta = (T[:, :-1] * a)[r, pl]
            rgb = torch.zeros(r1 - r0, 3, device="cuda", dtype=D).index_add(0, r, ta[:, None] * colour)
            rgba = torch.cat([rgb, 1.0 - T[:, -1:]], 1)
            img[idx[r0:r1]] = rgba.detach()
            if objective is not None:
                objective(idx[r0:r1], rgba, ta, facing, cell[k], r)
            r0 = r1
    if objective is not None:   # pixels outside a fisheye's circle stay black
        outside = torch.nonzero(~_directions(cam)[2]).flatten()
        objective(outside, img[outside], None, None, None)
    return img


def _exact_train(c, seed):
    params, cams, move, target, error = _train_inputs(c, seed)
    params["p"].add_(move, alpha=1.0)
    P = {k: v.to(D).requires_grad_(True) for k, v in params.items()}
    rays = _rays(cams)
    n = c["cells"]
    contribution, err = (torch.zeros(n, device="cuda", dtype=D) for _ in range(2))
    total, images, base = torch.zeros((), device="cuda", dtype=D), [], 0
    for cam in cams:
        def objective(idx, rgba, ta, facing, cell, r=None, base=base):
            nonlocal total
            v = ((rgba[:, :3] - target[base + idx].to(D)) ** 2).sum() / (3 * rays)
            if c["full"]:
                v = v + LAMBDA_SPARSE * rgba[:, 3].sum() / rays
                if ta is not None:
                    v = v + LAMBDA_NORMAL * (ta * facing).sum()
                    contribution.index_add_(0, cell, ta.detach())
                    err.index_add_(0, cell, ta.detach() * error[base + idx].to(D)[r])
            total = total + v.detach()
            if v.requires_grad:
                v.backward()

        images.append(_exact_view(P, cam, objective).reshape(cam.height, cam.width, 4))
        base += cam.width * cam.height
    if c["full"]:
        total = total + _exact_connect(P)
    out = {"images": images, "loss": total}
    if c["full"]:
        out["contribution"], out["error"] = contribution, err
    out["grads"] = {f: P[f].grad if P[f].grad is not None else torch.zeros_like(P[f]) for f in FIELDS}
    return out


def _exact_connect(P):
    total, n = 0.0, P["p"].shape[0]
    for a in range(0, n, 2048):
        i = torch.arange(a, min(n, a + 2048), device="cuda")
        with torch.no_grad():
            d2 = ((P["p"][i][:, None] - P["p"][None]) ** 2).sum(-1)
            ii, jj = torch.nonzero(d2 < (P["radius"][i][:, None] + P["radius"][None]) ** 2, as_tuple=True)
            ii = i[ii]
            ii, jj = ii[ii != jj], jj[ii != jj]
        ov = P["radius"][ii] + P["radius"][jj] - (P["p"][ii] - P["p"][jj]).norm(dim=1)
        v = LAMBDA_CONNECT * (ov.clamp(min=0.0) ** 2).sum()
        v.backward()
        total = total + v.detach()
    return total
