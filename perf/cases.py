"""The work that a user of the rasterizer has it do, as timed cases.

A case is a dict of plain values; ``listed()`` names the standing ones,
``draw(rng)`` gives one more of the same ranges.  ``prepare(case, seed)`` makes
what a program holds before the call (the map, the cameras, target images, a
captured graph), ``run(state)`` is one pass through the public entry points,
``work(case)`` the bytes and operations such a pass cannot do without, and
``exact(case, seed)`` the same results from plain torch in binary64.

Scenes follow the seeded workloads of the tests and the benchmark (a box in
front of one camera, a 20 x 20 x 4 m room seen by level or arbitrarily rotated
cameras, a 40 x 40 m lot with obstacles), drawn here on the GPU because inputs
are made many times.
"""
import math

import numpy as np
import torch

from paper_2409_18122_amd import raster

DEV = "cuda"
ROOM = ((-10.0, -10.0, 0.0), (10.0, 10.0, 4.0))
UNEVEN = ((160, 120), (320, 240), (640, 480))
T_MIN, A_MIN, A_MAX, Z_NEAR = 1e-4, float(np.float32(1.0 / 255.0)), float(np.float32(0.99)), float(np.float32(0.2))
T_MIN = float(np.float32(T_MIN))
GRADS = ("means", "log_scales", "quats", "opacity", "colors")


def listed():
    return [
        # one small preview of a sparse map: latency and launches decide
        {"name": "forward_128x96_2k", "kind": "forward", "n": 2000, "views": 1, "width": 128, "height": 96},
        # an odd-sized frame of a room-scale map, all four images, as a viewer asks for it
        {"name": "forward_1279x717_300k", "kind": "forward", "n": 300000, "views": 1, "width": 1279, "height": 717},
        # the mapper's iteration on the newest frame, captured once and replayed
        {"name": "map_graph_640x480_200k", "kind": "step", "api": "graph", "loss": "l1", "iso": False, "n": 200000,
         "views": 1, "width": 640, "height": 480},
        # the same iteration with the full loss (SSIM), call by call: the map changes size between iterations
        {"name": "map_eager_ssim_640x480_200k", "kind": "step", "api": "eager", "loss": "ssim", "iso": False,
         "n": 200000, "views": 1, "width": 640, "height": 480},
        # a torch training loop over two odd-sized frames of the paper's isotropic map, with an alpha term
        {"name": "autograd_iso_2x333x251_50k", "kind": "step", "api": "autograd", "loss": "l1", "iso": True, "n": 50000,
         "views": 2, "width": 333, "height": 251},
        # refinement over eight keyframes that share one map
        {"name": "map_graph_8x1280x720_1m", "kind": "step", "api": "graph", "loss": "l1", "iso": False, "n": 1000000,
         "views": 8, "width": 1280, "height": 720},
        # a planning step that scores a ring of candidate views once
        {"name": "score_64x320x240_500k", "kind": "score", "api": "eager", "mode": "rendered", "n": 500000, "views": 64,
         "width": 320, "height": 240},
        # a planner that scores hundreds of views of mixed sizes over and over on a large map
        {"name": "score_graph_256_uneven_2m", "kind": "score", "api": "graph", "mode": "rendered", "n": 2000000,
         "views": 256, "width": 0, "height": 0},
        # the paper's own view metric over 64 trajectories of 9 states, and their choice
        {"name": "utility_64x9_2m", "kind": "utility", "n": 2000000, "paths": 64, "steps": 9},
        # after each map update: the Gaussians' uncertainty and the regions' means
        {"name": "bookkeeping_2m", "kind": "bookkeeping", "n": 2000000, "size": 2.5, "squared": False},
        # one motion primitive against a lot-sized map (a planner expanding one node)
        {"name": "collision_1x129_3m", "kind": "collision", "n": 3000000, "paths": 1, "samples": 129, "clearance": True,
         "no_alloc": False},
        # a tree layer of 64 primitives against it
        {"name": "collision_64x129_3m", "kind": "collision", "n": 3000000, "paths": 64, "samples": 129,
         "clearance": True, "no_alloc": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("forward", "step", "step", "score", "score", "utility", "bookkeeping", "collision"))
    if kind == "forward":
        w = _log(rng, 64, 1280)
        return {"kind": kind, "n": _log(rng, 500, 500000), "views": rng.choice((1, 1, 3)), "width": w,
                "height": int(w * rng.uniform(0.5, 0.8))}
    if kind == "step":
        w = _log(rng, 96, 1280)
        return {"kind": kind, "api": rng.choice(("graph", "eager", "autograd")), "loss": rng.choice(("l1", "ssim")),
                "iso": rng.random() < 0.3, "n": _log(rng, 2000, 1000000), "views": rng.choice((1, 2, 4, 8)), "width": w,
                "height": int(w * rng.uniform(0.5, 0.75))}
    if kind == "score":
        w = rng.choice((0, 160, 320, rng.randrange(97, 320)))
        return {"kind": kind, "api": rng.choice(("graph", "eager")), "mode": rng.choice(("rendered", "binary")),
                "n": _log(rng, 20000, 2000000), "views": _log(rng, 4, 256), "width": w, "height": w * 3 // 4}
    if kind == "utility":
        return {"kind": kind, "n": _log(rng, 10000, 2000000), "paths": _log(rng, 1, 64), "steps": rng.choice((5, 9))}
    if kind == "bookkeeping":
        return {"kind": kind, "n": _log(rng, 10000, 3000000), "size": rng.choice((2.5, 1.0, 0.5)),
                "squared": rng.random() < 0.3}
    return {"kind": kind, "n": _log(rng, 10000, 3000000), "paths": _log(rng, 1, 64),
            "samples": rng.choice((129, 129, rng.randrange(17, 129))), "clearance": rng.random() < 0.7,
            "no_alloc": rng.random() < 0.25}


# ------------------------------------------------------------------ inputs


def _gen(seed):
    g = torch.Generator(DEV)
    g.manual_seed(seed)
    return g


def _map(gen, n, lo, hi, ls=(-3.0, 0.5), beta=False, iso=False, clusters=False):
    """A seeded map: planar float32 arrays as the library takes them."""
    u = lambda *s: torch.rand(*s, generator=gen, device=DEV)  # noqa: E731
    z = lambda *s: torch.randn(*s, generator=gen, device=DEV)  # noqa: E731
    lo, hi = torch.tensor(lo, device=DEV)[:, None], torch.tensor(hi, device=DEV)[:, None]
    g = {"means": lo + (hi - lo) * u(3, n), "log_scales": ls[0] + ls[1] * z(1 if iso else 3, n)}
    if not iso:
        q = z(4, n)
        g["quats"] = q / q.norm(dim=0, keepdim=True)
    # Beta(1/2, 1/2) is the arcsine distribution
    g["opacity"] = torch.sin(0.5 * math.pi * u(n)).square() if beta else torch.sigmoid(z(n))
    g["colors"], g["uncert"] = u(3, n), u(n)
    if clusters:  # the tenth nearest to eight centres is uncertain
        c = lo + (hi - lo) * u(3, 8)
        d2 = torch.stack([(g["means"] - c[:, k:k + 1]).square().sum(0) for k in range(8)]).amin(0)
        g["uncert"] = torch.where(d2 <= d2.kthvalue(max(1, n // 10)).values, torch.ones_like(d2), g["uncert"])
    return {k: v.float().contiguous() for k, v in g.items()}


def _camera(w, h, f, R, T):
    return {"width": w, "height": h, "fx": float(np.float32(f)), "fy": float(np.float32(f)), "cx": w / 2.0,
            "cy": h / 2.0, "R": np.asarray(R, np.float32).reshape(3, 3), "T": np.asarray(T, np.float32).reshape(3)}


def _level(x, y, z, yaw):
    c, s = math.cos(yaw), math.sin(yaw)
    return np.array([[s, 0.0, c], [-c, 0.0, s], [0.0, -1.0, 0.0]]), (x, y, z)


def _cameras(case, rng):
    """One camera on the box, level keyframes in the room, or (width 0) arbitrary views of mixed sizes."""
    w, h, n = case["width"], case["height"], case["views"]
    if case["kind"] != "score" and n == 1:
        return [_camera(w, h, 0.82 * w, np.eye(3), np.zeros(3))]
    cams = []
    for _ in range(n):
        if w:
            R, T = _level(*rng.uniform(-9.5, 9.5, 2), 1.0, rng.uniform(0.0, 2.0 * math.pi))
            cams.append(_camera(w, h, 0.82 * w, R, T))
            continue
        q, r = np.linalg.qr(rng.standard_normal((3, 3)))
        q = q * np.sign(np.diag(r))
        q[:, 0] *= np.sign(np.linalg.det(q))
        vw, vh = UNEVEN[rng.integers(3)]
        cams.append(_camera(vw, vh, 0.82 * vw, q, (*rng.uniform(-9.5, 9.5, 2), rng.uniform(0.2, 3.8))))
    return cams


def _targets(gen, cams):
    """Smooth RGB-D frames, packed view after view."""
    rgb, dep = [], []
    for c in cams:
        low = torch.rand(1, 4, 9, 12, generator=gen, device=DEV)
        im = torch.nn.functional.interpolate(low, (c["height"], c["width"]), mode="bilinear", align_corners=True)[0]
        im = (im + 0.02 * torch.randn(im.shape, generator=gen, device=DEV)).clamp(0.0, 1.0)
        rgb.append(im[:3].reshape(-1))
        dep.append(1.0 + 4.0 * im[3].reshape(-1))
    return torch.cat(rgb).contiguous(), torch.cat(dep).contiguous()


def _lot(gen, n):
    """A 40 x 40 m lot: 60 % on the ground, the rest on the mantles of 80 upright cylinders."""
    u = lambda k, lo, hi: lo + (hi - lo) * torch.rand(k, generator=gen, device=DEV)  # noqa: E731
    z = lambda k: 0.02 * torch.randn(k, generator=gen, device=DEV)  # noqa: E731
    ng = int(0.6 * n)
    nc = n - ng
    cx, cy, rad, hgt = u(80, -18, 18), u(80, -18, 18), u(80, 0.3, 2.0), u(80, 0.5, 3.0)
    k = torch.randint(80, (nc,), generator=gen, device=DEV)
    phi = u(nc, 0.0, 2.0 * math.pi)
    m = torch.stack([torch.cat([u(ng, -20, 20), cx[k] + rad[k] * phi.cos() + z(nc)]),
                     torch.cat([u(ng, -20, 20), cy[k] + rad[k] * phi.sin() + z(nc)]),
                     torch.cat([z(ng), u(nc, 0.0, 1.0) * hgt[k]])])
    ls = -3.5 + 0.3 * torch.randn(3, n, generator=gen, device=DEV)
    return {"means": m.float().contiguous(), "log_scales": ls.float().contiguous()}


def _arcs(rng, paths, samples):
    """Points on 5 m motion primitives half a metre above the ground, planar 3 x (paths samples)."""
    x0, th0, kap = rng.uniform(-17, 17, (2, paths, 1)), rng.uniform(0, 2 * math.pi, (paths, 1)), rng.uniform(-0.3, 0.3, (paths, 1))
    ds = 5.0 / max(samples - 1, 1)
    th = th0 + kap * np.arange(samples) * ds
    step = np.concatenate([np.zeros((paths, 1)), np.ones((paths, samples - 1)) * ds], 1)
    back = np.concatenate([th[:, :1], th[:, :-1]], 1)
    x, y = x0[0] + np.cumsum(step * np.cos(back), 1), x0[1] + np.cumsum(step * np.sin(back), 1)
    p = np.stack([x.ravel(), y.ravel(), np.full(x.size, 0.5)]).astype(np.float32)
    return torch.from_numpy(p).to(DEV).contiguous()


def _states(rng, paths, steps):
    """The level cameras along candidate trajectories, and their offsets."""
    cams = []
    for _ in range(paths):
        (x, y), th, kap = rng.uniform(-8.0, 8.0, 2), rng.uniform(0.0, 2.0 * math.pi), rng.uniform(-0.6, 0.6)
        for _ in range(steps):
            cams.append(_camera(320, 240, 262.5, *_level(x, y, 1.0, th)))
            x, y, th = x + 0.5 * math.cos(th), y + 0.5 * math.sin(th), th + 0.5 * kap
    return cams, torch.arange(paths + 1, device=DEV, dtype=torch.int32) * steps


def _inputs(case, seed):
    gen, rng, kind, n = _gen(seed), np.random.default_rng(seed), case["kind"], case["n"]
    if kind in ("forward", "step"):
        near = case["views"] == 1 and n <= 300000
        box = ((-5.0, -2.0, 2.0), (5.0, 2.0, 12.0)) if n > 5000 else ((-2.0, -2.0, 2.0), (2.0, 2.0, 6.0))
        g = _map(gen, n, *(box if near else ROOM), iso=case.get("iso", False))
        cams = _cameras(case, rng)
        if case["views"] == 1 and not near:
            cams = [_camera(case["width"], case["height"], 0.82 * case["width"], *_level(*rng.uniform(-9.5, 9.5, 2), 1.0, rng.uniform(0.0, 6.28)))]
        tgt = _targets(gen, cams) if kind == "step" else None
        return g, cams, tgt
    if kind == "score":
        uneven = not case["width"]
        return _map(gen, n, *ROOM, ls=(-3.5, 0.7) if uneven else (-3.0, 0.5), beta=uneven, clusters=True), _cameras(case, rng), None
    if kind == "utility":
        return (_map(gen, n, *ROOM, clusters=True), *_states(rng, case["paths"], case["steps"]))
    if kind == "bookkeeping":
        g = _map(gen, n, *ROOM)
        prev = g["means"] + 0.01 * torch.randn(3, n, generator=gen, device=DEV)
        prev[:, ::3] = g["means"][:, ::3]  # a third of the map was not seen by the update
        return g["means"], prev.contiguous(), g["uncert"]
    return _lot(gen, n), _arcs(rng, case["paths"], case["samples"]), None


_ctx = None


def _context():
    """The program's one library context."""
    global _ctx
    if _ctx is None:
        _ctx = raster.Context(0)
    return _ctx


def prepare(case, seed):
    kind, ctx = case["kind"], _context()
    s = {"case": case, "ctx": ctx, "in": _inputs(case, seed)}
    g = s["in"][0]
    if kind in ("forward", "step", "score"):
        s["S"] = dict(raster.DEFAULTS, isotropic=int(case.get("iso", False)))
    if kind == "step":
        cams, (t_rgb, t_dep) = s["in"][1:]
        s["grads"] = {k: torch.zeros_like(g[k]) for k in GRADS if k in g}
        if case["api"] == "graph":
            lam = {} if case["loss"] == "l1" else {"lambda1": 0.4, "lambda2": 0.1}
            s["graph"] = raster.MapGraph(ctx, g, cams, t_rgb, t_dep, 0.5 if case["loss"] == "l1" else 1.0, s["S"],
                                         grads=s["grads"], **lam)
    if kind == "score" and case["api"] == "graph":
        cams = s["in"][1]
        s["graph"] = raster.ScoreGraph(ctx, g, len(cams), max(c["width"] for c in cams), max(c["height"] for c in cams),
                                       s["S"], probe=cams, mode=case["mode"])
    if kind in ("score", "utility"):
        s["cams"] = raster.make_cameras(s["in"][1])
    return s


# --------------------------------------------------------------------- run


def run(s):
    case, ctx = s["case"], s["ctx"]
    return {"forward": _run_forward, "step": _run_step, "score": _run_score, "utility": _run_utility,
            "bookkeeping": _run_bookkeeping, "collision": _run_collision}[case["kind"]](s, case, ctx)


def _run_forward(s, case, ctx):
    g, cams, _ = s["in"]
    out, frame = raster.render(ctx, g, cams, s["S"])
    frame.close()
    return out


def _image_loss(rgb, dep, alpha, t_rgb, t_dep, p):
    """What a torch training loop computes on the images: L1 colour, depth and a silhouette term; p pixels a view."""
    return ((rgb - t_rgb).abs().sum() + 0.5 * (dep - t_dep).abs().sum() + 0.1 * (1.0 - alpha).square().sum()) / p


def _run_step(s, case, ctx):
    g, cams, (t_rgb, t_dep) = s["in"]
    if case["api"] == "autograd":
        leaf = {k: v.detach().requires_grad_(k in GRADS) for k, v in g.items()}
        rgb, dep, alpha, _ = raster.rasterize(ctx, leaf, cams, s["S"])
        loss = _image_loss(rgb, dep, alpha, t_rgb, t_dep, case["width"] * case["height"])
        loss.backward()
        return {"rgb": rgb.detach(), "depth": dep.detach(), "alpha": alpha.detach(), "grads": {k: leaf[k].grad for k in GRADS if k in g}}
    for t in s["grads"].values():
        t.zero_()
    if case["api"] == "graph":
        loss = s["graph"].launch()
        return {"loss": loss, "rgb": s["graph"].rgb, "depth": s["graph"].depth, "grads": s["grads"]}
    frame = raster.Frame(ctx, g, cams, s["S"])
    frame.bin_sort()
    out = frame.render(("rgb", "depth"))
    if case["loss"] == "l1":
        loss, d_rgb, d_dep = frame.loss(out["rgb"], out["depth"], t_rgb, t_dep)
    else:
        loss, d_rgb, d_dep = frame.loss_ssim(out["rgb"], out["depth"], t_rgb, t_dep)
    frame.backward(d_rgb, d_dep, grads=s["grads"])
    frame.close()
    return {"loss": loss, "rgb": out["rgb"], "depth": out["depth"], "grads": s["grads"]}


def _run_score(s, case, ctx):
    if case["api"] == "graph":
        return s["graph"].launch(s["cams"])
    return raster.score_views(ctx, s["in"][0], s["cams"], s["S"], mode=case["mode"])


def _run_utility(s, case, ctx):
    g, _, off = s["in"]
    lo_hi = raster.uncertainty_thresholds(ctx, g["uncert"])
    u = raster.view_utility(ctx, g, s["cams"], lo_hi)
    util, best = raster.trajectory_select(ctx, u["xi"], off)
    return {"lo_hi": lo_hi, **u, "utility": util, "best": best}


def _run_bookkeeping(s, case, ctx):
    cur, prev, u = s["in"]
    new = raster.uncertainty_update(ctx, prev, cur, u, squared=case["squared"])
    count, total, mean = raster.region_utility(ctx, cur, new, (*ROOM[0], *ROOM[1]), case["size"])
    return {"u": new, "count": count, "sum": total, "mean": mean}


def _run_collision(s, case, ctx):
    g, pts, _ = s["in"]
    hit, clear = raster.collision_check(ctx, g, pts, 0.25, 3.0, clearance=case["clearance"], no_alloc=case["no_alloc"])
    return {"hit": hit, "clearance": clear} if case["clearance"] else {"hit": hit}


# -------------------------------------------------------------------- work


def work(case):
    """Each input read once, each output written once; a pixel of these maps takes about 250 contributing splats
    before it is opaque (fewer on a sparse map), at 36, 72 and 28 floating-point operations each forward, backward
    and scored (a fused multiply-add counts as two)."""
    kind, n = case["kind"], case["n"]
    if kind in ("forward", "step", "score"):
        pix = case["views"] * (case["width"] * case["height"] or sum(a * b for a, b in UNEVEN) / 3)
        pairs = pix * 250.0 * min(1.0, n / 50000.0)
        if kind == "score":
            return {"bytes": 48.0 * n + 8.0 * case["views"], "flops": 28.0 * pairs}
        if kind == "forward":
            return {"bytes": 60.0 * n + 24.0 * pix, "flops": 36.0 * pairs}
        return {"bytes": 2 * 56.0 * n + 32.0 * pix, "flops": 108.0 * pairs}
    if kind == "utility":
        return {"bytes": 16.0 * n, "flops": 30.0 * n * case["paths"] * case["steps"]}
    if kind == "bookkeeping":
        return {"bytes": 32.0 * n, "flops": 12.0 * n}
    # a point needs its nearest Gaussians only, the map one pass
    return {"bytes": 24.0 * n + 20.0 * case["paths"] * case["samples"], "flops": 10.0 * n}


# ------------------------------------------------------------------- exact
# Plain torch in binary64: projection, front-to-back compositing in blocks of
# pixels over the depth-ordered splats whose support box meets the block, and
# autograd for the gradients.


def _project64(g, cam, iso):
    """The visible splats of one camera in depth order: (fields that carry gradients, boxes, uncertainty)."""
    W, H = cam["width"], cam["height"]
    R = torch.tensor(cam["R"], dtype=torch.float64, device=DEV)
    t = R.T @ (g["means"] - torch.tensor(cam["T"], dtype=torch.float64, device=DEV)[:, None])
    ok = (t[2] > Z_NEAR) & (g["opacity"] >= A_MIN)
    idx = ok.nonzero()[:, 0]
    t, o = t[:, idx], g["opacity"][idx]
    iz = 1.0 / t[2]
    mx, my = cam["fx"] * t[0] * iz + cam["cx"], cam["fy"] * t[1] * iz + cam["cy"]
    if iso:
        r = g["log_scales"][0, idx].exp()
        sxx, syy = (cam["fx"] * r * iz).square(), (cam["fy"] * r * iz).square()
        sxy = torch.zeros_like(sxx)
    else:
        w, x, y, z = g["quats"][:, idx] / g["quats"][:, idx].norm(dim=0, keepdim=True)
        Q = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y), 2 * (x * y + w * z),
                         1 - 2 * (x * x + z * z), 2 * (y * z - w * x), 2 * (x * z - w * y), 2 * (y * z + w * x),
                         1 - 2 * (x * x + y * y)]).view(3, 3, -1)
        A = torch.einsum("ka,kbn->abn", R, Q) * g["log_scales"][:, idx].exp()[None]
        b0 = cam["fx"] * iz * (A[0] - t[0] * iz * A[2])
        b1 = cam["fy"] * iz * (A[1] - t[1] * iz * A[2])
        sxx, sxy, syy = (b0 * b0).sum(0), (b0 * b1).sum(0), (b1 * b1).sum(0)
    det = sxx * syy - sxy * sxy
    with torch.no_grad():
        rho2 = 2.0 * torch.log(o / A_MIN)
        hx, hy = (rho2 * sxx).sqrt(), (rho2 * syy).sqrt()
        box = torch.stack([(mx - hx).ceil().clamp(min=0), (mx + hx).floor().clamp(max=W - 1),
                           (my - hy).ceil().clamp(min=0), (my + hy).floor().clamp(max=H - 1)])
        keep = ((det > 0) & (box[0] <= box[1]) & (box[2] <= box[3])).nonzero()[:, 0]
        keep = keep[t[2, keep].float().sort(stable=True).indices]  # binary32 depth, ties by index
    f = torch.stack([mx, my, syy / det, -sxy / det, sxx / det, o, *g["colors"][:, idx], t[2]])[:, keep]
    return f, box[:, keep], g["uncert"][idx[keep]] if "uncert" in g else None


def _composite64(f, unc, px, py, binary=False):
    """r, g, b, depth, alpha, uncertainty (6 x pixels) of the given pixels; f: depth-ordered splat fields."""
    T = torch.ones_like(px)
    live = torch.ones_like(px, dtype=torch.bool)
    out = torch.zeros(6, px.numel(), dtype=torch.float64, device=DEV)
    for at in range(0, f.shape[1], 256):
        c, u = f[:, at:at + 256], unc[at:at + 256]
        dx, dy = px[:, None] - c[0], py[:, None] - c[1]
        a = c[5] * torch.exp(-0.5 * (c[2] * dx * dx + 2.0 * c[3] * dx * dy + c[4] * dy * dy))
        a = torch.where(a > A_MAX, torch.full_like(a, A_MAX), a)
        a = torch.where(a >= A_MIN, a, torch.zeros_like(a))
        after = T[:, None] * (1.0 - a).cumprod(1)
        with torch.no_grad():
            go = live[:, None] & (after >= T_MIN)
        w = torch.where(go, a * torch.cat([T[:, None], after[:, :-1]], 1), torch.zeros_like(a))
        out = out + torch.cat([c[6:] @ w.T, w.sum(1)[None], (((go & (a > 0)).double() if binary else w) @ u)[None]])
        T = after[:, -1]
        live = go[:, -1]
        if not bool(live.any()):
            break
    return out


def _blocks(cam, f, box, unc, edge=64):
    """(pixel indices, their coordinates, the splats that can reach them) block by block."""
    W, H = cam["width"], cam["height"]
    for y0 in range(0, H, edge):
        row = ((box[2] <= y0 + edge - 1) & (box[3] >= y0)).nonzero()[:, 0]
        for x0 in range(0, W, edge):
            sel = row[(box[0, row] <= x0 + edge - 1) & (box[1, row] >= x0)]
            ys, xs = torch.meshgrid(torch.arange(y0, min(y0 + edge, H), device=DEV), torch.arange(x0, min(x0 + edge, W), device=DEV), indexing="ij")
            ys, xs = ys.reshape(-1), xs.reshape(-1)
            yield ys * W + xs, xs.double(), ys.double(), sel


def _render64(g, cams, iso, binary=False):
    """Per view: the projected splats and the 6 x P images."""
    for cam in cams:
        f, box, unc = _project64(g, cam, iso)
        with torch.no_grad():
            fd, unc = f.detach(), torch.zeros(f.shape[1], dtype=torch.float64, device=DEV) if unc is None else unc.detach()
            img = torch.zeros(6, cam["width"] * cam["height"], dtype=torch.float64, device=DEV)
            for pix, px, py, sel in _blocks(cam, fd, box, unc):
                if sel.numel():
                    img[:, pix] = _composite64(fd[:, sel], unc[sel], px, py, binary)
        yield cam, f, box, unc, img


def _ssim64(x, y):
    k = torch.exp(-torch.arange(-5, 6, dtype=torch.float64, device=DEV).square() / 4.5)
    k = k / k.sum()
    blur = lambda v: torch.nn.functional.conv2d(torch.nn.functional.conv2d(v[:, None], k.view(1, 1, 1, 11), padding=(0, 5)),  # noqa: E731
                                                k.view(1, 1, 11, 1), padding=(5, 0))[:, 0]
    mx, my = blur(x), blur(y)
    sx, sy, sxy = blur(x * x) - mx * mx, blur(y * y) - my * my, blur(x * y) - mx * my
    return (((2 * mx * my + 1e-4) * (2 * sxy + 9e-4)) / ((mx * mx + my * my + 1e-4) * (sx + sy + 9e-4))).mean()


def _exact_step(case, seed):
    g32, cams, (t_rgb, t_dep) = _inputs(case, seed)
    g = {k: v.double().requires_grad_(k in GRADS) for k, v in g32.items()}
    images, total, at = [], 0.0, 0
    for cam, f, box, unc, img in _render64(g, cams, case["iso"]):
        W, H = cam["width"], cam["height"]
        p = W * H
        tr, td = t_rgb[3 * at:3 * (at + p)].double().view(3, p), t_dep[at:at + p].double()
        at += p
        im = img.clone().requires_grad_()
        if case["api"] == "autograd":
            loss = _image_loss(im[:3], im[3], im[4], tr, td, p)
        elif case["loss"] == "l1":
            loss = ((im[:3] - tr).abs().sum() + 0.5 * (im[3] - td).abs().sum()) / p
        else:
            loss = ((im[3] - td).abs().sum() + 0.4 * (im[:3] - tr).abs().sum()) / p + 0.1 * (1.0 - _ssim64(im[:3].view(3, H, W), tr.view(3, H, W)))
        loss.backward()
        total = total + loss.detach()
        leaf = f.detach().requires_grad_()
        for pix, px, py, sel in _blocks(cam, leaf, box, unc):
            if sel.numel():
                _composite64(leaf[:, sel], unc[sel], px, py).backward(im.grad[:, pix])
        f.backward(leaf.grad)
        images.append(img)
    grads = {k: g[k].grad for k in GRADS if k in g}
    flat = lambda a, b: torch.cat([i[a:b].reshape(-1) for i in images])  # noqa: E731
    if case["api"] == "autograd":
        return {"rgb": flat(0, 3), "depth": flat(3, 4), "alpha": flat(4, 5), "grads": grads}
    return {"loss": total.reshape(1), "rgb": flat(0, 3), "depth": flat(3, 4), "grads": grads}


def _exact_utility(case, seed):
    g, cams, off = _inputs(case, seed)
    u, m = g["uncert"].double(), g["means"].double()
    sd = (u - u.mean()).square().mean().sqrt()
    lo, hi = u.mean() - 0.5 * sd, u.mean() + 0.5 * sd
    high, low, rows = (u > hi).double(), (u < lo).double(), []
    for c in cams:
        t = torch.tensor(c["R"], dtype=torch.float64, device=DEV).T @ (m - torch.tensor(c["T"], dtype=torch.float64, device=DEV)[:, None])
        x, y = c["fx"] * t[0] / t[2] + c["cx"], c["fy"] * t[1] / t[2] + c["cy"]
        v = ((t[2] > Z_NEAR) & (t[2] <= 5.0) & (x >= 0) & (x <= c["width"] - 1) & (y >= 0) & (y <= c["height"] - 1)).double()
        rows.append(torch.stack([(high * v).sum(), (low * v).sum(), (u * v).sum()]))
    r = torch.stack(rows, 1)
    xi = r[0] - r[1]
    return {"lo_hi": torch.stack([lo, hi]), "n_high": r[0].long(), "n_low": r[1].long(), "sum_u": r[2], "xi": xi,
            "utility": xi.view(case["paths"], case["steps"]).sum(1), "best": None}


def _exact_bookkeeping(case, seed):
    cur, prev, u = _inputs(case, seed)
    d2 = (cur.double() - prev.double()).square().sum(0)
    new = torch.where((cur == prev).all(0), u.double(), d2 if case["squared"] else d2.sqrt())
    lo, hi = torch.tensor(ROOM[0], dtype=torch.float64, device=DEV), torch.tensor(ROOM[1], dtype=torch.float64, device=DEV)
    dims = ((hi - lo) / case["size"]).ceil().long()
    cell = ((cur.double() - lo[:, None]) / case["size"]).floor().long()
    inside = ((cell >= 0) & (cell < dims[:, None])).all(0)
    r = (cell[0] + dims[0] * (cell[1] + dims[1] * cell[2]))[inside]
    count = torch.bincount(r, minlength=int(dims.prod()))
    # the regions sum the stored binary32 values
    total = torch.zeros(count.numel(), dtype=torch.float64, device=DEV).index_add_(0, r, new.float().double()[inside])
    return {"u": new, "count": count, "sum": total, "mean": torch.where(count > 0, total / count.clamp(min=1), torch.zeros_like(total))}


def _exact_collision(case, seed):
    g, pts, _ = _inputs(case, seed)
    m, r = g["means"].double(), 3.0 * g["log_scales"].double().amax(0).exp()
    hit, clear = [], []
    for at in range(0, pts.shape[1], 32):
        p = pts[:, at:at + 32].double()
        d2 = sum((p[k][:, None] - m[k]).square() for k in range(3))
        hit.append((d2 < (0.25 + r).square()).any(1).int())
        clear.append((d2.sqrt() - r).amin(1))
    return {"hit": torch.cat(hit), "clearance": torch.cat(clear)} if case["clearance"] else {"hit": torch.cat(hit)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "forward":
        g, cams, _ = _inputs(case, seed)
        img = [v[4] for v in _render64({k: v.double() for k, v in g.items()}, cams, False)]
        flat = lambda a, b: torch.cat([i[a:b].reshape(-1) for i in img])  # noqa: E731
        return {"rgb": flat(0, 3), "depth": flat(3, 4), "alpha": flat(4, 5), "unc": flat(5, 6)}
    if kind == "score":
        g, cams, _ = _inputs(case, seed)
        g = {k: v.double() for k, v in g.items()}
        return torch.stack([v[4][5].sum() for v in _render64(g, cams, False, case["mode"] == "binary")])
    return {"step": _exact_step, "utility": _exact_utility, "bookkeeping": _exact_bookkeeping, "collision": _exact_collision}[kind](case, seed)
