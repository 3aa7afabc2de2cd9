"""Workloads of the rasterizer for performance measurement.

Each case is one call (or one iteration) that a Gaussian-SLAM program makes
through this package's public entry points, at the sizes of the repository's
own configurations (64x48, 640x480 and 1200x680 frames; 1,000 to 1,000,000
Gaussians) and at odd ones between them:

  frame   a small differentiable render: forward, L1 loss, backward to the
          parameters and the pose
  view    a forward render alone (an alpha mask for seeding, a novel view)
  grad    a mapping iteration that leaves the gradients to the caller
  map     a whole mapping iteration: L1 + SSIM colour, depth, scale
          regulariser, backward with Adam fused in
  refine  a colour-refinement iteration of the merged map
  batch   a mapping iteration over several keyframes at once
  track   one tracking iteration issued call by call
  graph   tracking of one frame as a captured graph
  seed    seeding from a keyframe: candidates and their neighbour queries
  upkeep  new Gaussians from the kept points, and opacity pruning of the map
          with the optimiser's moments
  train   a training step of the tracking initialiser
  propose one proposal of the tracking initialiser

Scenes are views of the procedural room of `synth`, made on the GPU: Gaussians
back-projected from noisy depth, scales from the nearest-neighbour distance
that this sampling density gives. `exact` repeats a case in float64 with plain
torch operations.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2312_10070_amd import gsr, initnet, synth

DEV = "cuda"
GROUPS = gsr.PARAM_GROUPS
# Adam step sizes late in a schedule (a hundredth of the first iterations' 1e-4, 5e-5, 1e-3, 1e-3, 2.5e-3)
LRS = {"means": 1e-6, "scales": 5e-7, "quats": 1e-5, "opacities": 1e-5, "colors": 2.5e-5}
ADAM_STEP, GRAD_SCALE = 200, 1e-6
LAMBDA_SSIM, LAMBDA_REG = 0.2, 1.0
LAMBDA_C, INLIER = 0.5, 50.0
NET_LR = 2e-6
SEED_P = 600_000 / (1200 * 680)  # uniform candidates per pixel of a first keyframe


# ---- cases -------------------------------------------------------------------

def listed():
    return [
        # the smallest differentiable render: unit tests, a thumbnail; launches and host work are all of it
        dict(name="frame_64x48_1k", kind="frame", width=64, height=48, n=1000),
        # the image a keyframe is seeded against, from a grown sub-map
        dict(name="view_1200x680_1M", kind="view", width=1200, height=680, n=1_000_000),
        # mapping with the caller's own optimiser, at a size that no tile shape divides
        dict(name="grad_801x533_200k", kind="grad", width=801, height=533, n=200_001, deterministic=False),
        # the paper's mapping iteration on a Replica-sized frame: what a SLAM run spends most of its time on
        dict(name="map_1200x680_500k", kind="map", width=1200, height=680, n=500_000),
        # post-processing of the merged map, frames of the tracking camera
        dict(name="refine_640x480_300k", kind="refine", width=640, height=480, n=300_000),
        # the active sub-map against all its keyframes: the largest call
        dict(name="batch_8x1200x680_1M", kind="batch", width=1200, height=680, n=1_000_000, views=8,
             blocks_per_cu=8, tile_w=16, tile_h=16),
        # a tracking iteration of a program that keeps the loop on the host
        dict(name="track_640x480_500k", kind="track", width=640, height=480, n=500_000),
        # frame-to-model tracking, the other half of a SLAM run (a short frame of 20 iterations)
        dict(name="graph_640x480_500k", kind="graph", width=640, height=480, n=500_000, iters=20),
        # a new sub-map's first keyframe: 600,000 uniform and the edge candidates of 816,000 pixels
        dict(name="seed_1200x680_500k", kind="seed", width=1200, height=680, n=500_000, first=True),
        # the map's upkeep around a keyframe's iterations: points added, low opacities pruned
        dict(name="upkeep_500k", kind="upkeep", n=500_000, points=100_000, thre=0.5),
        # training of the tracking initialiser
        dict(name="train_b64", kind="train", batch=64),
        # its use on a frame: packing and one forward
        dict(name="propose_640x480", kind="propose", width=640, height=480),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "view", "grad", "grad", "map", "map", "refine", "batch", "track", "graph", "seed",
                       "upkeep", "train", "propose"])
    if kind == "upkeep":
        n = _log_uniform(rng, 1000, 500_000)
        return dict(kind=kind, n=n, points=max(1, int(n * rng.uniform(0.01, 0.5))), thre=rng.choice([0.1, 0.5]))
    if kind == "train":
        return dict(kind=kind, batch=rng.randint(1, 64))
    if kind == "propose":
        f = rng.randint(1, 7)
        return dict(kind=kind, width=160 * f, height=120 * f)
    w = _log_uniform(rng, 48, 160) if kind == "frame" else _log_uniform(rng, 160, 1200)
    h = max(36, min(680, int(w * rng.uniform(0.5, 0.8))))
    most = {"view": 1_000_000, "batch": 400_000}.get(kind, 500_000)
    n = max(500, min(most, int(w * h * math.exp(rng.uniform(math.log(0.1), math.log(1.6))))))
    c = dict(kind=kind, width=w, height=h, n=n)
    if kind == "grad":
        c["deterministic"] = rng.random() < 0.2
    if kind == "batch":
        c["views"] = rng.randint(2, 5)
        c["blocks_per_cu"] = rng.choice([0, 4, 8])
        c["tile_w"], c["tile_h"] = rng.choice([(16, 16), (16, 16), (32, 8), (8, 32)])
    if kind == "graph":
        c["iters"] = rng.randint(5, 20)
    if kind == "seed":
        c["first"] = rng.random() < 0.5
    return c


# ---- inputs ------------------------------------------------------------------

def _camera(case):
    w, h = case["width"], case["height"]
    f = {1200: 600.0, 640: 525.0, 64: 60.0}.get(w, 0.6 * w)
    return synth.Intrinsics(w, h, f, f, w / 2.0, h / 2.0)


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _rand(gen, *shape):
    return torch.rand(*shape, device=DEV, dtype=torch.float64, generator=gen)


def _randn(gen, *shape):
    return torch.randn(*shape, device=DEV, dtype=torch.float64, generator=gen)


def _raycast(room, cam, pose7, xy):
    """Depth, colour and world points of the room along the rays of the pixels xy [m,2]."""
    R, t = synth.pose7_to_Rt(pose7)
    T = lambda a: torch.as_tensor(np.asarray(a), device=DEV, dtype=torch.float64)
    d = torch.stack([(xy[:, 0] - cam.cx) / cam.fx, (xy[:, 1] - cam.cy) / cam.fy, torch.ones_like(xy[:, 0])], 1) @ T(R)
    c = T(-R.T @ t)
    lo, hi = T(synth.ROOM_MIN), T(synth.ROOM_MAX)
    # the walls: the far side of the room's box
    far = torch.where(d > 0, (hi - c) / d, (lo - c) / d)
    best, axis = far.min(1)
    surf = 2 * axis + (d.gather(1, axis[:, None])[:, 0] > 0).long()
    for b in range(len(room.boxes_min)):
        t0, t1 = (T(room.boxes_min[b]) - c) / d, (T(room.boxes_max[b]) - c) / d
        tn, ax = torch.minimum(t0, t1).max(1)
        hit = (tn <= torch.maximum(t0, t1).min(1)[0]) & (tn > 1e-6) & (tn < best)
        best, surf, axis = torch.where(hit, tn, best), torch.where(hit, 6 + b, surf), torch.where(hit, ax, axis)
    p = c + best[:, None] * d
    u, v = p.gather(1, ((axis + 1) % 3)[:, None])[:, 0], p.gather(1, ((axis + 2) % 3)[:, None])[:, 0]
    ph = T(room.phase)[surf]
    check = 0.08 * (((torch.floor(u / 0.1) + torch.floor(v / 0.1)) % 2) * 2 - 1)
    s1, s2 = 0.06 * torch.sin(2 * math.pi * u / 0.37 + ph[:, 0]), 0.06 * torch.sin(2 * math.pi * v / 0.23 + ph[:, 1])
    col = T(room.base_colors)[surf] + check[:, None] + s1[:, None] * T([1.0, 0.6, 0.2]) + s2[:, None] * T([0.2, 0.5, 1.0])
    return best, col.clamp(0, 1), p


def _frame(room, cam, pose7, gen, holes=0.0):
    """An RGB-D frame of the room with a sensor's noise (and a share of pixels without depth)."""
    y, x = torch.meshgrid(torch.arange(cam.height, device=DEV), torch.arange(cam.width, device=DEV), indexing="ij")
    d, c, _ = _raycast(room, cam, pose7, torch.stack([x.reshape(-1), y.reshape(-1)], 1).double())
    c = (c + 0.01 * _randn(gen, *c.shape)).clamp(0, 1)
    d = d * (1 + 0.003 * _randn(gen, *d.shape))
    if holes:
        d = torch.where(_rand(gen, d.shape[0]) < holes, 0.0, d)
    return (c.t().reshape(3, cam.height, cam.width).float().contiguous(),
            d.reshape(cam.height, cam.width).float().contiguous())


def _gaussians(room, cam, views, n, gen, optimised):
    """n Gaussians back-projected from the views. Their scale is the nearest-neighbour distance of points that
    are Poisson on the surface (in each view's pixels) and off it by the depth noise. `optimised`: opacities as a
    mapping run leaves them instead of the initial 0.5."""
    per = [n // len(views) + (i < n % len(views)) for i in range(len(views))]
    means, cols, lat = [], [], []
    for pose, m in zip(views, per):
        xy = torch.stack([_rand(gen, m) * cam.width - 0.5, _rand(gen, m) * cam.height - 0.5], 1)
        d, col, _ = _raycast(room, cam, pose, xy)
        d = d + 0.005 * _randn(gen, m)
        R, t = synth.pose7_to_Rt(pose)
        pc = torch.stack([(xy[:, 0] - cam.cx) / cam.fx * d, (xy[:, 1] - cam.cy) / cam.fy * d, d], 1)
        means.append((pc - torch.as_tensor(t, device=DEV)) @ torch.as_tensor(R, device=DEV))
        cols.append(col)
        lat.append(d / cam.fx)
    means, cols, px = torch.cat(means), torch.cat(cols), torch.cat(lat)
    r2 = torch.cumsum(-torch.log(1 - _rand(gen, n, 12)), 1) * (cam.width * cam.height / (math.pi * n)) * (px * px)[:, None]
    nn = (r2 + (0.005 * math.sqrt(2) * _randn(gen, n, 12)) ** 2).min(1)[0].sqrt()
    q = _randn(gen, n, 4)
    g = dict(means=means, scales=nn[:, None] * torch.exp(0.3 * _randn(gen, n, 3)),
             quats=q / q.norm(dim=1, keepdim=True),
             opacities=torch.sigmoid(0.3 + 0.8 * _randn(gen, n)) if optimised else torch.full((n,), 0.5, device=DEV),
             colors=cols)
    return {k: v.float().contiguous() for k, v in g.items()}


def _pose(p7):
    return torch.as_tensor(np.asarray(p7, np.float32), device=DEV)


def _scene(case, seed, n_views, optimised, holes=0.0, off=(0.0, 0.0)):
    """Room, camera, Gaussians, a pose near the seeding views and the frame seen from the base view."""
    cam, rng, gen = _camera(case), np.random.default_rng(seed), _gen(seed)
    room = synth.make_room(seed)
    base = synth.open_view(room, rng, cam)
    views = [base] + [synth.perturb_pose(base, rng, rng.uniform(0, 0.3), rng.uniform(0, 10)) for _ in range(n_views - 1)]
    g = _gaussians(room, cam, views, case["n"], gen, optimised)
    color, depth = _frame(room, cam, base, gen, holes)
    pose = synth.perturb_pose(base, rng, *off) if off != (0.0, 0.0) else base
    return dict(g=g, cam=cam, camera=gsr.camera_from(cam), pose=_pose(pose), color=color, depth=depth, gen=gen, room=room)


def _moments(g, gen):
    m = {k: (GRAD_SCALE * torch.randn(v.shape, device=DEV, generator=gen)) for k, v in g.items()}
    v = {k: GRAD_SCALE ** 2 * (0.5 + torch.rand(x.shape, device=DEV, generator=gen)) for k, x in g.items()}
    return m, v


def _net_frames(case, seed):
    """Packed-size frames for the initialiser: a render-like image and the frame seen 2 cm / 1 degree off."""
    cam, rng, gen = _camera(case), np.random.default_rng(seed), _gen(seed)
    room = synth.make_room(seed)
    base = synth.open_view(room, rng, cam)
    near = synth.perturb_pose(base, rng, 0.02, 1.0)
    return (*_frame(room, cam, near, gen), *_frame(room, cam, base, gen))


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case, kind=kind)
    if kind in ("frame", "grad", "view", "refine"):
        s |= _scene(case, seed, {"frame": 1, "grad": 1}.get(kind, 5), kind in ("view", "refine"))
        s["opts"] = gsr.RasterOpts(deterministic=int(case.get("deterministic", False)))
        if kind == "refine":
            m, v = _moments({"colors": s["g"]["colors"]}, s["gen"])
            s |= dict(m=m["colors"], v=v["colors"])
    elif kind == "map":
        s |= _scene(case, seed, 1, False)
        s["m"], s["v"] = _moments(s["g"], s["gen"])
    elif kind in ("track", "graph"):
        s |= _scene(case, seed, 5, True, holes=0.03, off=(0.02, 1.0))
        if kind == "graph":
            g = tuple(s["g"][k] for k in GROUPS)
            _, _, _, st = gsr.render_fwd(*g, s["pose"], s["camera"])
            K = gsr.state_stats(st)["K"]
            st.release()
            s["graph"] = gsr.TrackGraph(*g, s["camera"], s["color"], s["depth"], n_iters=case["iters"],
                                        lambda_c=LAMBDA_C, inlier_mult=INLIER, K_cap=max(4096, 3 * K // 2))
            s["losses"] = torch.empty(case["iters"], device=DEV)
    elif kind == "batch":
        cam, rng, gen = _camera(case), np.random.default_rng(seed), _gen(seed)
        room = synth.make_room(seed)
        lo, size = synth.ROOM_MIN, synth.ROOM_MAX - synth.ROOM_MIN
        spot, yaw = rng.uniform(lo + 0.3 * size, lo + 0.7 * size), rng.uniform(-np.pi, np.pi)

        def view(move, turn):
            d = rng.normal(size=3)
            return synth.camera_pose(spot + move * rng.uniform() * d / np.linalg.norm(d), yaw + turn,
                                     np.deg2rad(rng.uniform(-10, 10)))

        g = _gaussians(room, cam, [view(0.4, np.deg2rad(rng.uniform(-25, 25))) for _ in range(16)], case["n"], gen, False)
        keys = [view(0.3, np.deg2rad(a) * rng.choice([-1, 1])) for a in np.linspace(10, 90, case["views"])]
        frames = [_frame(room, cam, p, gen) for p in keys]
        s |= dict(g=g, cam=cam, camera=gsr.camera_from(cam), poses=torch.stack([_pose(p) for p in keys]),
                  color=torch.stack([f[0] for f in frames]), depth=torch.stack([f[1] for f in frames]),
                  opts=gsr.RasterOpts(tile_w=case["tile_w"], tile_h=case["tile_h"]))
    elif kind == "seed":
        s |= _scene(case, seed, 5, True, holes=0.03, off=(0.1, 5.0))
        h, w = s["depth"].shape
        # later keyframes: the part of the frame that the sub-map does not cover, with a soft border
        x = torch.arange(w, device=DEV, dtype=torch.float32) / w
        s["alpha"] = None if case["first"] else (1.6 * x + 0.1 * torch.rand((h, w), device=DEV, generator=s["gen"])).clamp(0, 1)
        # random numbers that choose the same number of pixels for every seed
        open_ = (s["depth"] > 0) if case["first"] else (s["depth"] > 0) & (s["alpha"] < 0.6)
        share = 0.71 if case["first"] else 0.2
        rank = torch.where(open_, torch.rand((h, w), device=DEV, generator=s["gen"]), 2.0).reshape(-1).argsort()
        u = SEED_P + 0.25 + (0.75 - SEED_P) * torch.rand(h * w, device=DEV, generator=s["gen"])
        m = int(share * h * w)
        u[rank[:m]] = SEED_P * 0.999 * torch.rand(m, device=DEV, generator=s["gen"])
        s["u"] = u.reshape(h, w).contiguous()
    elif kind == "upkeep":
        gen, n, m = _gen(seed), case["n"], case["points"]
        s["points"], s["rgb"] = (torch.rand((m, 3), device=DEV, generator=gen) for _ in range(2))
        s["nn"] = (0.01 + 0.04 * torch.rand(m, device=DEV, generator=gen)) ** 2
        s["keep"] = (torch.rand(m, device=DEV, generator=gen).argsort() < m // 3).int()
        g = {k: torch.rand((n, w) if w > 1 else (n,), device=DEV, generator=gen) for k, w in zip(GROUPS, (3, 3, 4, 1, 3))}
        # the same opacities for every seed, in another order
        q = ((torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) / n)
        g["opacities"] = torch.sigmoid(1.0 + 1.5 * torch.special.ndtri(q)).float()[torch.rand(n, device=DEV, generator=gen).argsort()].contiguous()
        s["g"] = g
        s["m"], s["v"] = _moments(g, gen)
    elif kind == "train":
        b, gen, rng = case["batch"], _gen(seed), np.random.default_rng(seed)
        s["net"] = gsr.InitNet(max_batch=64)
        s["net"].set_params(torch.from_numpy(initnet.init_params(int(seed))).to(DEV))
        x = torch.nn.functional.interpolate(torch.rand((b, 8, 15, 20), device=DEV, generator=gen), (120, 160), mode="bilinear")
        x[:, 4:] = 0.4 * (x[:, 4:] - 0.5)
        s["x"] = (x + 0.02 * torch.randn(x.shape, device=DEV, generator=gen)).permute(0, 2, 3, 1).contiguous().bfloat16()
        s["labels"] = torch.from_numpy(np.stack([initnet.random_twist(rng) for _ in range(b)]).astype(np.float32)).to(DEV)
        s["scale"] = torch.tensor(initnet.LABEL_SCALE, device=DEV)
    elif kind == "propose":
        s["net"] = gsr.InitNet(max_batch=1)
        s["net"].set_params(torch.from_numpy(initnet.init_params(int(seed))).to(DEV))
        s["frames"] = _net_frames(case, seed)
        s["x"] = torch.empty((1, 120, 160, 8), device=DEV, dtype=torch.bfloat16)
    else:
        raise ValueError(f"unknown kind {kind}")
    return s


# ---- one pass ----------------------------------------------------------------

def run(s):
    kind, case = s["kind"], s["case"]
    g = s.get("g")
    if kind in ("frame", "grad"):
        c, d, a, st = gsr.render_fwd(*(g[k] for k in GROUPS), s["pose"], s["camera"], s["opts"])
        loss, gc, gd = gsr.loss_l1(c, d, s["color"], s["depth"])
        grads = gsr.render_bwd(st, gc, gd, None, want_params=True, want_pose=kind == "frame")
        st.release()
        return dict(color=c, depth=d, alpha=a, loss=loss, grads=grads)
    if kind == "view":
        c, d, a, st = gsr.render_fwd(*(g[k] for k in GROUPS), s["pose"], s["camera"], s["opts"])
        st.release()
        return dict(color=c, depth=d, alpha=a)
    if kind == "map":
        c, d, _, st = gsr.render_fwd(*(g[k] for k in GROUPS), s["pose"], s["camera"])
        loss, gc, gd = gsr.loss_map(c, d, s["color"], s["depth"], lam=LAMBDA_SSIM)
        gsr.loss_reg(g["scales"], LAMBDA_REG, loss)
        gsr.render_bwd_adam(st, gc, gd, s["m"], s["v"], LRS, ADAM_STEP, scale_reg=LAMBDA_REG)
        st.release()
        return dict(loss=loss, params=g, m=s["m"], v=s["v"])
    if kind == "refine":
        c, d, _, st = gsr.render_fwd(*(g[k] for k in GROUPS), s["pose"], s["camera"])
        loss, gc, gd = gsr.loss_map(c, d, s["color"], s["depth"], lam=LAMBDA_SSIM, w_color=1.0, w_depth=0.0)
        grads = gsr.render_bwd(st, gc, gd, None, want_params=True, want_pose=False, groups=("colors",))
        st.release()
        gsr.adam_step(g["colors"], s["m"], s["v"], grads["colors"], ADAM_STEP, LRS["colors"])
        return dict(loss=loss, grad=grads["colors"], colors=g["colors"], m=s["m"], v=s["v"])
    if kind == "batch":
        c, d, a, st = gsr.render_fwd_batch(*(g[k] for k in GROUPS), s["poses"], s["camera"], s["opts"],
                                           blocks_per_cu=case["blocks_per_cu"])
        loss, gc, gd = gsr.loss_l1(c, d, s["color"], s["depth"])
        grads = gsr.render_bwd(st, gc, gd, None, want_params=True, want_pose=False)
        st.release()
        return dict(color=c, depth=d, alpha=a, loss=loss, grads=grads)
    if kind == "track":
        c, d, a, st = gsr.render_fwd(*(g[k] for k in GROUPS), s["pose"], s["camera"])
        loss, gc, gd, med = gsr.loss_track(c, d, a, s["color"], s["depth"], LAMBDA_C, INLIER)
        grads = gsr.render_bwd(st, gc, gd, None, want_params=False, want_pose=True)
        st.release()
        return dict(color=c, depth=d, alpha=a, loss=loss, median=med, grads=grads)
    if kind == "graph":
        return dict(pose=s["graph"].run(s["pose"].clone(), s["losses"]), losses=s["losses"])
    if kind == "seed":
        pts, cols = gsr.seed_candidates(s["color"], s["depth"], s["u"], s["pose"], s["camera"], SEED_P,
                                        0.25 if case["first"] else 0.0, 0.05, s["alpha"], 0.6)
        nn, keep = gsr.seed_query(g["means"], pts, 0.01, 0.05)
        return dict(points=pts, colors=cols, nn_d2=nn, keep=keep)
    if kind == "upkeep":
        new = gsr.seed_gaussians(s["points"], s["rgb"], s["nn"], s["keep"])
        n, p, m, v = gsr.prune(g, case["thre"], s["m"], s["v"])
        return dict(new=new, n=n, params=p, m=m, v=v)
    if kind == "train":
        net, b = s["net"], case["batch"]
        net.set_input(s["x"])
        out = net.forward(b)
        loss = net.backward(b, s["labels"], s["scale"])
        net.adam(NET_LR)
        params, grads = net.get_params(with_grads=True)
        return dict(out=out, loss=loss, params=params, grads=grads)
    if kind == "propose":
        gsr.pack_rgbd_pair(*s["frames"], s["x"][0], initnet.DEPTH_SCALE)
        return dict(x=s["x"], twist=initnet.predict(s["net"], s["x"]))
    raise ValueError(f"unknown kind {kind}")


# ---- work --------------------------------------------------------------------

def work(case):
    """Bytes: every input read and every output written once. Operations: per pixel about 72 support-box pairs
    (15 operations to evaluate) and 55 composited ones (12 forward, 48 more backward) where the sub-map is as dense
    as half the pixels or more, as counted on such frames; 390 per pixel and channel for SSIM."""
    kind, n, px = case["kind"], case.get("n", 0), case.get("width", 0) * case.get("height", 0)
    views = case.get("views", 1)
    dense = px * views * min(1.0, 2.0 * n / max(px, 1)) if px else 0.0
    fwd = dense * (72 * 15 + 55 * 12)
    bwd = dense * (72 * 15 + 55 * 48)
    b_fwd, b_params, b_loss = 56 * n + 20 * px * views, 56 * n, 16 * px * views
    net = 2 * 9 * (8 * 64 * 4800 + 64 * 64 * (1200 + 300 + 80))  # one image's convolutions forward
    n_net = initnet.layout()[1]
    return {
        "frame": lambda: dict(bytes=b_fwd + b_loss + b_params, flops=fwd + bwd),
        "view": lambda: dict(bytes=b_fwd, flops=fwd),
        "grad": lambda: dict(bytes=b_fwd + b_loss + b_params, flops=fwd + bwd),
        "map": lambda: dict(bytes=b_loss + 6 * b_params, flops=fwd + bwd + 3 * 390 * px),
        "refine": lambda: dict(bytes=56 * n + 12 * px + 72 * n, flops=fwd + bwd + 3 * 390 * px),
        "batch": lambda: dict(bytes=b_fwd + b_loss + b_params, flops=fwd + bwd),
        "track": lambda: dict(bytes=b_fwd + b_loss, flops=fwd + bwd),
        "graph": lambda: dict(bytes=56 * n + b_loss, flops=case["iters"] * (fwd + bwd)),
        "seed": lambda: dict(bytes=20 * px + 12 * n + 0.75 * px * (24 + 8), flops=0.75 * px * 465 * 8),
        "upkeep": lambda: dict(bytes=(1 + 0.7) * 168 * n + case["points"] * (36 + 56 / 3), flops=n),
        "train": lambda: dict(bytes=case["batch"] * 120 * 160 * 16 + 28 * n_net, flops=3 * case["batch"] * net),
        "propose": lambda: dict(bytes=32 * px + 120 * 160 * 16 + 4 * n_net, flops=net),
    }[kind]()


# ---- the same in float64 ------------------------------------------------------

AMIN, AMAX, TMIN, GUARD, LOWPASS, SLACK = 1.0 / 255.0, 0.99, 1e-4, 1.3, 0.3, 1e-3
BLOCK = 32  # pixels of a block's edge


def _rotation(q):
    w, x, y, z = (q / q.norm(dim=-1, keepdim=True)).unbind(-1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], -1).reshape(*q.shape[:-1], 3, 3)


def _project64(p, pose, cam):
    """Screen-space rows [k, 10] (u, v, conic a, b, c, opacity, r, g, b, z) of the Gaussians that reach the
    image, their indices and pixel boxes."""
    R = _rotation(pose[:4])
    x = p["means"] @ R.t() + pose[4:]
    with torch.no_grad():
        near = torch.nonzero((x[:, 2] > cam.near_z) & (p["opacities"] >= AMIN))[:, 0]
    x, op = x[near], p["opacities"][near]
    M = _rotation(p["quats"][near]) * p["scales"][near][:, None, :]
    RM = R @ M
    z = x[:, 2]
    lx, ly = GUARD * max(cam.cx, cam.width - cam.cx) / cam.fx, GUARD * max(cam.cy, cam.height - cam.cy) / cam.fy
    X, Y = (x[:, 0] / z).clamp(-lx, lx), (x[:, 1] / z).clamp(-ly, ly)
    r0 = (cam.fx / z)[:, None] * (RM[:, 0] - X[:, None] * RM[:, 2])  # rows of J R M
    r1 = (cam.fy / z)[:, None] * (RM[:, 1] - Y[:, None] * RM[:, 2])
    sxx, sxy, syy = (r0 * r0).sum(1) + LOWPASS, (r0 * r1).sum(1), (r1 * r1).sum(1) + LOWPASS
    det = sxx * syy - sxy * sxy
    rows = torch.stack([cam.fx * x[:, 0] / z + cam.cx, cam.fy * x[:, 1] / z + cam.cy, syy / det, -sxy / det, sxx / det, op,
                        *p["colors"][near].unbind(1), z], 1)
    with torch.no_grad():
        s = torch.log(op / AMIN) * (1 + SLACK) + SLACK
        ex, ey = torch.sqrt(2 * s * sxx), torch.sqrt(2 * s * syy)
        box = torch.stack([torch.ceil(rows[:, 0] - ex).clamp(min=0), torch.floor(rows[:, 0] + ex).clamp(max=cam.width - 1),
                           torch.ceil(rows[:, 1] - ey).clamp(min=0), torch.floor(rows[:, 1] + ey).clamp(max=cam.height - 1)], 1).long()
        seen = torch.nonzero((box[:, 0] <= box[:, 1]) & (box[:, 2] <= box[:, 3]))[:, 0]
    return rows[seen], near[seen], box[seen]


def _block_lists(rows, box, cam):
    """Row indices per block, nearest first: (indices, offsets of the blocks on the host)."""
    nbx, nby = -(-cam.width // BLOCK), -(-cam.height // BLOCK)
    order = torch.argsort(rows[:, 9].detach(), stable=True)
    b = box[order] // BLOCK
    wx, wy = b[:, 1] - b[:, 0] + 1, b[:, 3] - b[:, 2] + 1
    cnt = wx * wy
    rep = torch.repeat_interleave(torch.arange(len(order), device=DEV), cnt)
    k = torch.arange(len(rep), device=DEV) - (torch.cumsum(cnt, 0) - cnt)[rep]
    tile = (b[rep, 2] + k // wx[rep]) * nbx + b[rep, 0] + k % wx[rep]
    tile, at = torch.sort(tile, stable=True)
    ends = torch.cumsum(torch.bincount(tile, minlength=nbx * nby), 0).tolist()
    return order[rep[at]], [0] + ends, nbx


def _block64(r, x0, y0, x1, y1):
    """Colour, depth and alpha [pixels, 5] of one block from its rows."""
    y, x = torch.meshgrid(torch.arange(y0, y1, device=DEV), torch.arange(x0, x1, device=DEV), indexing="ij")
    dx, dy = x.reshape(-1, 1) - r[:, 0], y.reshape(-1, 1) - r[:, 1]
    raw = r[:, 5] * torch.exp(-0.5 * (r[:, 2] * dx * dx + r[:, 4] * dy * dy) - r[:, 3] * dx * dy)
    a = raw.clamp(max=AMAX)
    a = torch.where(a >= AMIN, a, torch.zeros_like(a))
    logT = torch.cumsum(torch.log1p(-a), 1)
    w = torch.where(torch.exp(logT) >= TMIN, a * torch.exp(logT - torch.log1p(-a)), torch.zeros_like(a))
    return torch.cat([w @ r[:, 6:10], w.sum(1, keepdim=True)], 1)


def _render64(rows, box, cam, up=None):
    """The image [5, H, W], or, given the upstream gradients [5, H, W], the gradient of the rows."""
    ids, ends, nbx = _block_lists(rows, box, cam)
    out = torch.zeros((5, cam.height, cam.width), device=DEV, dtype=torch.float64)
    grad = torch.zeros_like(rows)
    rows = rows.detach()
    for t in range(len(ends) - 1):
        if ends[t] == ends[t + 1]:
            continue
        y0, x0 = BLOCK * (t // nbx), BLOCK * (t % nbx)
        y1, x1 = min(y0 + BLOCK, cam.height), min(x0 + BLOCK, cam.width)
        idx = ids[ends[t]:ends[t + 1]]
        if up is None:
            out[:, y0:y1, x0:x1] = _block64(rows[idx], x0, y0, x1, y1).t().reshape(5, y1 - y0, x1 - x0)
        else:
            r = rows[idx].requires_grad_(True)
            with torch.enable_grad():
                o = _block64(r, x0, y0, x1, y1)
            grad.index_add_(0, idx, torch.autograd.grad(o, r, up[:, y0:y1, x0:x1].reshape(5, -1).t())[0])
    return out if up is None else grad


def _ssim64(x, y):
    k = torch.exp(-(torch.arange(11, device=DEV, dtype=torch.float64) - 5) ** 2 / 4.5)
    k = k / k.sum()
    f = lambda t: torch.nn.functional.conv2d(torch.nn.functional.conv2d(t[:, None], k.view(1, 1, 11, 1), padding=(5, 0)),
                                             k.view(1, 1, 1, 11), padding=(0, 5))[:, 0]
    mx, my = f(x), f(y)
    vx, vy, cxy = f(x * x) - mx * mx, f(y * y) - my * my, f(x * y) - mx * my
    return ((2 * mx * my + 1e-4) * (2 * cxy + 9e-4) / ((mx * mx + my * my + 1e-4) * (vx + vy + 9e-4))).mean()


def _loss64(kind, img, color, depth):
    """(loss, the median where there is one) of the image [5, H, W]."""
    c, d, a = img[:3], img[3], img[4]
    if kind == "track":
        e = (d - depth).abs()
        valid = depth > 0
        med = e[valid].detach().median() if valid.any() else e.new_zeros(())
        w = torch.where(valid & (e <= INLIER * med), a ** 3, torch.zeros_like(a)).detach()
        return (w * (LAMBDA_C * (c - color).abs().sum(0) + (1 - LAMBDA_C) * e)).sum(), med.reshape(1)
    lam = LAMBDA_SSIM if kind in ("map", "refine") else 0.0
    loss = (1 - lam) * (c - color).abs().mean()
    if lam:
        loss = loss + lam * (1 - _ssim64(c, color))
    return loss + (0.0 if kind == "refine" else (d - depth).abs().mean()), None


def _adam64(p, m, v, g, lr):
    m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
    return p - lr * (m / (1 - 0.9 ** ADAM_STEP)) / ((v / (1 - 0.999 ** ADAM_STEP)).sqrt() + 1e-8), m, v


def _exact_render(s):
    kind, cam = s["kind"], s["cam"]
    p = {k: s["g"][k].double().requires_grad_(True) for k in GROUPS}
    poses = (s["poses"] if kind == "batch" else s["pose"][None]).double()
    tc, td = s["color"].double(), s["depth"].double()
    if kind != "batch":
        tc, td = tc[None], td[None]
    V = len(poses)
    images, loss, med, gpose = [], 0.0, None, None
    for i in range(V):
        pose = poses[i].clone().requires_grad_(True)
        rows, _, box = _project64(p, pose, cam)
        with torch.no_grad():
            images.append(_render64(rows, box, cam))
        if kind == "view":
            continue
        img = images[-1].clone().requires_grad_(True)
        one, med = _loss64(kind, img, tc[i], td[i])
        one = one / V
        loss = loss + one.detach()
        up = torch.autograd.grad(one, img)[0]
        up[4] = 0  # no loss here has a gradient for alpha
        rows.backward(_render64(rows, box, cam, up))
        gpose = pose.grad
    out = torch.stack(images)
    grads = {k: v.grad if v.grad is not None else torch.zeros_like(v) for k, v in p.items()}
    res = dict(color=out[:, :3], depth=out[:, 3], alpha=out[:, 4]) if kind == "batch" else \
        dict(color=out[0, :3], depth=out[0, 3], alpha=out[0, 4])
    if kind == "view":
        return res
    loss = loss.reshape(1)
    if kind in ("frame", "track"):
        R, t = _rotation(poses[0][:4]), poses[0][4:]
        gq, gt = gpose[:4], gpose[4:]
        # the left perturbation (rho, phi): q' = (1, phi / 2) q, t' = t + rho + phi x t, at a unit q
        n = poses[0][:4].norm()
        w, x, y, z = (poses[0][:4] / n).unbind()
        dq = 0.5 * torch.stack([torch.stack([-x, w, -z, y]), torch.stack([-y, z, w, -x]), torch.stack([-z, -y, x, w])])
        twist = torch.cat([gt, dq @ (gq * n) + torch.linalg.cross(t, gt)])
        pg = dict(pose7=gpose, twist6=twist)
    if kind == "track":
        return res | dict(loss=loss, median=med, grads=pg)
    if kind in ("frame", "grad", "batch"):
        return res | dict(loss=loss, grads=grads | (pg if kind == "frame" else {}))
    if kind == "refine":
        c, m, v = _adam64(p["colors"].detach(), s["m"].double(), s["v"].double(), grads["colors"], LRS["colors"])
        return dict(loss=loss, grad=grads["colors"], colors=c, m=m, v=v)
    # map: the regulariser joins the loss and the scale gradient
    sc = p["scales"].detach().requires_grad_(True)
    reg = LAMBDA_REG * (sc - sc.mean(1, keepdim=True)).abs().sum() / sc.shape[0]
    grads["scales"] = grads["scales"] + torch.autograd.grad(reg, sc)[0]
    new = {k: _adam64(p[k].detach(), s["m"][k].double(), s["v"][k].double(), grads[k], LRS[k]) for k in GROUPS}
    return dict(loss=loss + reg.detach(), params={k: v[0] for k, v in new.items()}, m={k: v[1] for k, v in new.items()},
                v={k: v[2] for k, v in new.items()})


def _exact_seed(s):
    """Points of the chosen pixels and their colours; the nearest neighbours are left out (a float32 minimum over the
    same float32 points)."""
    cam, pose = s["cam"], s["pose"].double()
    y, x = torch.nonzero((s["depth"] > 0) & (s["u"] < SEED_P), as_tuple=True)
    z = s["depth"][y, x].double()
    pc = torch.stack([(x - cam.cx) * z / cam.fx, (y - cam.cy) * z / cam.fy, z], 1)
    return dict(points=(pc - pose[4:]) @ _rotation(pose[:4]), colors=s["color"][:, y, x].t().double(), nn_d2=None, keep=None)


def _exact_net(flat, x, labels=None, scale=None):
    w = {k: torch.as_tensor(v, device=DEV).requires_grad_(True) for k, v in initnet.to_oihw(flat).items()}
    a = x.double().permute(0, 3, 1, 2)
    for l in range(4):
        a = torch.relu(torch.nn.functional.conv2d(a, w[f"w{l}"], w[f"b{l}"], stride=2, padding=1))
    h, k = a.shape[2:]
    my = ((2 * torch.arange(h, device=DEV, dtype=torch.float64) + 1) / h - 1).view(1, 1, h, 1)
    mx = ((2 * torch.arange(k, device=DEV, dtype=torch.float64) + 1) / k - 1).view(1, 1, 1, k)
    pool = torch.cat([a.mean((2, 3)), (a * mx).mean((2, 3)), (a * my).mean((2, 3))], 1)
    out = pool @ w["wfc"].t() + w["bfc"]
    if labels is None:
        return out.detach()
    loss = 0.5 * (((out - labels.double()) / scale.double()) ** 2).sum() / len(x)
    loss.backward()
    return out.detach(), loss.detach().reshape(1), initnet.pack_grads_oihw({k: v.grad.cpu().numpy() for k, v in w.items()})


def exact(case, seed):
    kind = case["kind"]
    if kind == "graph":
        return None  # iterations of an optimiser: small differences grow
    s = prepare(case, seed)
    if kind == "upkeep":
        keep = s["g"]["opacities"] >= case["thre"]
        pick = lambda t: {k: v[keep].double() for k, v in t.items()}
        j = s["keep"] != 0
        one = torch.ones(int(j.sum()), device=DEV, dtype=torch.float64)
        new = dict(means=s["points"][j].double(), colors=s["rgb"][j].double(), opacities=0.5 * one,
                   scales=s["nn"][j].double().sqrt()[:, None].expand(-1, 3),
                   quats=torch.stack([one, 0 * one, 0 * one, 0 * one], 1))
        return dict(new=new, n=int(keep.sum()), params=pick(s["g"]), m=pick(s["m"]), v=pick(s["v"]))
    if kind == "seed":
        return _exact_seed(s)
    if kind in ("train", "propose"):
        flat = initnet.init_params(int(seed))
        if kind == "train":
            out, loss, g = _exact_net(flat, s["x"], s["labels"], s["scale"])
            g = torch.as_tensor(g, device=DEV)
            return dict(out=out, loss=loss, grads=g, params=None)  # a first Adam step goes by the gradient's sign
        rc, rd, oc, od = (t.double() for t in s["frames"])
        r = torch.cat([rc, rd[None] * initnet.DEPTH_SCALE])
        o = torch.cat([oc, od[None] * initnet.DEPTH_SCALE])
        x = torch.nn.functional.avg_pool2d(torch.cat([r, 4.0 * (o - r)])[None], case["width"] // 160).permute(0, 2, 3, 1)
        return dict(x=x, twist=_exact_net(flat, x))
    return _exact_render(s)
