"""What the rasterizer is timed on: the work of a mapping back-end, through the
package's public entry points, over the range it is used in.

A case names a path (`kind`), the Gaussian pool (count, SH degree, geometry)
and the views.  The sizes are those of the repository's own workloads: one
128x96 view of 2,000 Gaussians up to 16 views of 1200x680 over 2 million.

kinds
  map       one mapping iteration as a captured graph: projection, binning,
            forward, loss, backward, Adam (what runs thousands of times)
  pose      one eager iteration that returns the gradients and the camera
            tangent for given image gradients (pose refinement)
  schedule  one step of the keyframe-scheduled loop: selection on the host,
            ids to the device, replay of the gathered graph, losses read back
  autograd  rasterize() and torch.autograd's backward through it
  render    rasterize() without gradients (evaluation, novel views)
  densify   clone / split / prune, then the spatial order of the new pool
  sort      the stand-alone sort of (key, value) pairs
"""
import functools
import math
import random

import numpy as np
import torch
import torch.nn.functional as F

import paper_2410_00486_amd as gsr
from paper_2410_00486_amd import _lib as L

DEV = "cuda"
FIELDS = ("means", "log_scales", "quats", "opacity_logits", "sh")
# learning rates of a map that has been optimised for a while (the schedule's
# end, a hundredth of its beginning), so that repeated passes stay on one scene
LRS = {"means": 1.6e-6, "log_scales": 5e-5, "quats": 1e-5, "opacity_logits": 5e-4, "sh": 2.5e-5}
BETA1, BETA2, EPS, STEP = 0.9, 0.999, 1e-15, 400
# scale of the carried Adam moments, per group (the gradients of an L1 mean)
MOMENT = {"means": 1e-5, "log_scales": 1e-6, "quats": 1e-6, "opacity_logits": 1e-6, "sh": 1e-6}
LAMBDA_DEPTH, LAMBDA_SSIM, LAMBDA_O = 0.1, 0.2, 0.01


def _case(name, kind, n, **kw):
    base = dict(name=name, kind=kind, n=n, deg=3, scene="room", views="", log_scale=-4.5, faint=0.0,
                tile="8x8", splat=True, radix=False, ordered=False, depth=True, ssim=False, reg=False)
    base.update(kw)
    return base


def listed():
    return [
        # the smallest differentiable call: a sketch of a scene, all defaults
        _case("autograd_slab_128x96", "autograd", 2_000, deg=0, scene="slab", views="slab:128x96",
              log_scale=-3.0, tile="16x16", splat=False),
        # the smallest mapping step: a young map, one small keyframe
        _case("map_slab_128x96", "map", 2_000, deg=0, scene="slab", views="slab:128x96", log_scale=-3.0,
              depth=False),
        # pose refinement of one RGB-D frame
        _case("pose_640x480_150k", "pose", 150_000, views="in:640x480"),
        # the ordinary mapping step: one keyframe of a room
        _case("map_1200x680_300k", "map", 300_000, views="in:1200x680", reg=True),
        # the same with the full loss (SSIM)
        _case("map_ssim_1200x680_300k", "map", 300_000, views="in:1200x680", ssim=True),
        # a differentiable call on a whole room with the entry point's defaults
        _case("autograd_1200x680_300k", "autograd", 300_000, views="over:1200x680", tile="16x16",
              splat=False),
        # evaluation of a map at four held-out views
        _case("render_4x1200x680_500k", "render", 500_000,
              views="in:1200x680,over:1200x680,in:1200x680,over:1200x680", tile="16x16", splat=False),
        # the scheduled loop: 4 of 16 keyframes of one RGB-D camera a step
        _case("schedule_4of16_640x480", "schedule", 300_000, views=",".join(["in:640x480"] * 16),
              radix=True, ordered=True, batch=4),
        # keyframes of several cameras, close-ups and overviews, one batch
        _case("map_8mixed_500k", "map", 500_000, radix=True, ordered=True,
              views="close:640x480,over:640x480,close:640x480,over:640x480,close:640x480,over:640x480,"
                    "close:1200x680,over:320x240"),
        # the large batch: 16 keyframes over a map of four rooms
        _case("map_16x1200x680_2M", "map", 2_000_000, scene="rooms", views=",".join(["in:1200x680"] * 16),
              log_scale=-5.0, faint=0.3, radix=True, ordered=True),
        # what the mapping loop does every few hundred iterations
        _case("densify_300k", "densify", 300_000),
        # the stand-alone sort at the size of a view's pairs
        _case("sort_1M_46bit", "sort", 1 << 20, bits=46),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["map", "map", "map", "map", "pose", "autograd", "autograd", "render", "schedule",
                       "densify", "sort"])
    if kind == "sort":
        return _pure(_case("", kind, _log_int(rng, 1_000, 4_000_000), bits=rng.randint(20, 62)))
    n = _log_int(rng, 2_000, 1_000_000)
    if kind == "densify":
        return _pure(_case("", kind, n, deg=rng.choice([0, 3, 3]), log_scale=_fill(n, 1)))
    one = kind in ("pose", "autograd")
    count = 1 if one else rng.choice([1, 1, 2, 3, 4, 6, 8, 12])
    wide = _log_int(rng, 100, 1200)
    size = "%dx%d" % (wide, max(64, int(wide * rng.uniform(0.55, 0.8))))
    views = []
    for _ in range(12 if kind == "schedule" else count):
        views.append("%s:%s" % (rng.choice(["in", "in", "over", "close"]), size))
        if kind in ("map", "render") and rng.random() < 0.5:  # keyframes of several cameras
            wide = _log_int(rng, 100, 1200)
            size = "%dx%d" % (wide, max(64, int(wide * rng.uniform(0.55, 0.8))))
    kw = dict(deg=rng.choice([0, 1, 2, 3, 3, 3]), views=",".join(views), log_scale=_fill(n, 1),
              faint=rng.choice([0.0, 0.0, 0.3]))
    if kind in ("autograd", "render"):
        kw.update(tile=rng.choice(["16x16", "16x16", "8x8"]), splat=False)
    else:
        batch = kind == "schedule" or count > 1
        kw.update(tile=rng.choice(["8x8", "8x8", "8x8", "16x8", "16x16"]), splat=rng.random() < 0.8,
                  radix=batch and rng.random() < 0.8, ordered=rng.random() < 0.5)
    if kind == "map":
        kw.update(depth=rng.random() < 0.8, ssim=rng.random() < 0.2, reg=rng.random() < 0.3)
    if kind == "schedule":
        kw.update(batch=rng.randint(1, 6))
    return _pure(_case("", kind, n, **kw))


def _pure(c):
    c.pop("name")
    return c


def _fill(n, rooms):
    """Log-scale at which n Gaussians cover the surfaces as 300k of -4.5 do."""
    return round(min(-2.5, max(-5.0, -4.5 + 0.5 * math.log(300_000 * rooms / n))), 3)


# ---------------------------------------------------------------- inputs

def _views(case):
    out = []
    for v in case["views"].split(","):
        where, size = v.split(":")
        out.append((where, *(int(x) for x in size.split("x"))))
    return out


def _tile(case):
    return tuple(int(x) for x in case["tile"].split("x"))


def _rooms(case):
    return [(6.0 * x, 5.0 * y) for y in range(2) for x in range(2)] if case["scene"] == "rooms" else [(0.0, 0.0)]


def _faces(rng, x0, y0):
    """A 6x5x3 m room with 20 boxes: (origin, edge, edge) of every rectangle."""
    ex, ey, ez = (6.0, 0, 0), (0, 5.0, 0), (0, 0, 3.0)
    o = (x0, y0, 0.0)
    faces = [(o, ex, ey), ((x0, y0, 3.0), ex, ey), (o, ex, ez), ((x0, y0 + 5.0, 0), ex, ez), (o, ey, ez),
             ((x0 + 6.0, y0, 0), ey, ez)]
    for _ in range(20):
        w, d, h = (rng.uniform(0.2, 1.2) for _ in range(3))
        yaw = rng.uniform(0, 2 * math.pi)
        a, b = np.array([math.cos(yaw), math.sin(yaw), 0.0]) * w, np.array([-math.sin(yaw), math.cos(yaw), 0.0]) * d
        c = np.array([x0 + rng.uniform(0.5, 5.5), y0 + rng.uniform(0.5, 4.5), 0.0]) - 0.5 * (a + b)
        z = np.array([0.0, 0.0, h])
        faces += [(c + z, a, b), (c, a, z), (c + b, a, z), (c, b, z), (c + a, b, z)]
    return faces


def _camera(rng, where, w, h, x0, y0):
    """A 20-float record: fx fy cx cy | R[9] | t[3] | near | bg[3]."""
    f, roll = (525.0 * w / 640 if w <= 640 else w / 2.0), rng.gauss(0, 0.05)
    if where == "slab":  # identity pose in front of the slab
        return [100.0, 100.0, w / 2, h / 2, 1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0, 0.2, 0, 0, 0]
    if where == "in":
        pos = np.array([x0 + rng.uniform(1, 5), y0 + rng.uniform(1, 4), rng.uniform(1.2, 1.8)])
        yaw, pitch = rng.uniform(0, 2 * math.pi), rng.gauss(0, 0.15)
        fwd = np.array([math.cos(yaw) * math.cos(pitch), math.sin(yaw) * math.cos(pitch), math.sin(pitch)])
    elif where == "over":  # from an upper corner over the room
        pos = np.array([x0 + rng.choice([0.3, 5.7]), y0 + rng.choice([0.3, 4.7]), 2.6])
        fwd = np.array([x0 + 3.0, y0 + 2.5, 0.6]) - pos + np.array([rng.gauss(0, 0.1) for _ in range(3)])
        f = w / 2.0
    else:  # close to a wall
        d, z, f = rng.uniform(0.4, 0.8), rng.uniform(0.8, 2.0), w / 2.0
        u, wall = rng.uniform(1, 4), rng.randrange(4)
        pos = np.array([[x0 + u, y0 + d, z], [x0 + u, y0 + 5 - d, z], [x0 + d, y0 + u, z], [x0 + 6 - d, y0 + u, z]][wall])
        fwd = np.array([[0, -1.0, 0], [0, 1.0, 0], [-1.0, 0, 0], [1.0, 0, 0]][wall])
        fwd = fwd + np.array([rng.gauss(0, 0.05) for _ in range(3)])
    fwd = fwd / np.linalg.norm(fwd)
    right = np.cross(fwd, [0.0, 0.0, 1.0])
    right /= np.linalg.norm(right)
    down = np.cross(fwd, right)
    right, down = math.cos(roll) * right + math.sin(roll) * down, -math.sin(roll) * right + math.cos(roll) * down
    R = np.stack([right, down, fwd])
    return [f, f, w / 2, h / 2, *R.reshape(-1), *(-R @ pos), 0.2, 0.0, 0.0, 0.0]


def _pool(case, seed):
    """Parameters (float32, on the GPU) in no spatial order."""
    rng = random.Random(seed)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    n, k = case["n"], (case["deg"] + 1) ** 2
    rand = lambda *s: torch.rand(*s, generator=gen, device=DEV)
    randn = lambda *s: torch.randn(*s, generator=gen, device=DEV)
    if case["scene"] == "slab":
        means = rand(n, 3) * 2 - 1 + torch.tensor([0.0, 0.0, 3.0], device=DEV)
    else:
        faces = [f for x0, y0 in _rooms(case) for f in _faces(rng, x0, y0)]
        o, u, v = (torch.tensor(np.array([f[i] for f in faces], np.float32), device=DEV) for i in range(3))
        area = torch.linalg.norm(torch.linalg.cross(u.double(), v.double()), dim=1).cumsum(0)
        at = torch.searchsorted((area / area[-1]).float(), rand(n)).clamp_(max=len(faces) - 1)
        means = o[at] + rand(n, 1) * u[at] + rand(n, 1) * v[at] + 0.01 * randn(n, 3)
    scales = case["log_scale"] + (0.5 if case["faint"] else 0.4 if case["scene"] != "slab" else 0.3) * randn(n, 3)
    quats = randn(n, 4)
    quats = quats / quats.norm(dim=1, keepdim=True)
    logits = randn(n)
    if case["faint"]:
        o = 0.001 + 0.049 * rand(n)
        logits = torch.where(rand(n) < case["faint"], torch.log(o / (1 - o)), logits)
    sh = 0.05 * randn(n, k, 3)
    sh[:, 0] = (rand(n, 3) - 0.5) / 0.28209479177387814
    return [x.float().contiguous() for x in (means, scales, quats, logits, sh)]


def _inputs(case, seed):
    """Everything a pass reads, from the seed alone: float32 tensors."""
    rng = random.Random(seed + 1)
    gen = torch.Generator(device=DEV).manual_seed(seed + 1)
    views, rooms = _views(case), _rooms(case)
    cams = torch.tensor(np.array([_camera(rng, wh, w, h, *rooms[i * len(rooms) // len(views)])
                                  for i, (wh, w, h) in enumerate(views)], np.float32), device=DEV)
    rgb, dep = [], []
    for _, w, h in views:  # smooth pictures with a little noise
        low = torch.rand(1, 4, h // 32 + 2, w // 32 + 2, generator=gen, device=DEV)
        img = F.interpolate(low, size=(h, w), mode="bilinear", align_corners=True)[0]
        rgb.append((0.9 * img[:3] + 0.1 * torch.rand(3, h, w, generator=gen, device=DEV)).reshape(-1))
        dep.append((0.5 + 4.0 * img[3]).reshape(-1))
    d = dict(views=views, wh=[(w, h) for _, w, h in views], cams=cams, params=_pool(case, seed),
             rgb=torch.cat(rgb).contiguous(), dep=torch.cat(dep).contiguous())
    if case["kind"] in ("pose", "autograd"):
        px = sum(w * h for w, h in d["wh"])
        d["gc"] = torch.randn(3 * px, generator=gen, device=DEV) / px
        d["gd"] = torch.randn(px, generator=gen, device=DEV) / px
    if case["kind"] in ("map", "schedule"):
        d["m"] = [0.3 * MOMENT[f] * torch.randn(x.shape, generator=gen, device=DEV)
                  for f, x in zip(FIELDS, d["params"])]
        d["v"] = [MOMENT[f] ** 2 * torch.exp(torch.randn(x.shape, generator=gen, device=DEV))
                  for f, x in zip(FIELDS, d["params"])]
    return d


def _densify_inputs(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed + 2)
    n = case["n"]
    p = _pool(case, seed)
    m = [1e-6 * torch.randn(x.shape, generator=gen, device=DEV) for x in p]
    v = [1e-12 * torch.rand(x.shape, generator=gen, device=DEV) for x in p]
    # a tenth has faded, an eighth each is selected as large (split) and as
    # small (cloned), all over the pool; some were not seen at all
    role = torch.randperm(n, generator=gen, device=DEV) % 40
    p[3] = torch.where(role < 4, -5.0 - p[3].abs(), p[3].clamp(min=-3.0))
    p[1] = torch.where(((role >= 4) & (role < 9))[:, None], p[1].clamp(min=-2.5), p[1].clamp(max=-3.0))
    chosen = (role >= 4) & (role < 14)
    seen = torch.randint(0, 20, (n,), generator=gen, device=DEV).float()
    seen = torch.where(chosen, seen + 1, seen)
    rate = torch.rand(n, generator=gen, device=DEV)
    accum = seen * torch.where(chosen, 1.2e-3 + 2e-3 * rate, 8e-4 * rate)
    normals = torch.randn(n, 2, 3, generator=gen, device=DEV)
    return p, m, v, accum.contiguous(), seen, normals


def _sort_inputs(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    n, bits = case["n"], case["bits"]
    keys = torch.randint(0, 1 << bits, (n,), generator=gen, device=DEV, dtype=torch.int64)
    at, k = torch.randperm(n, generator=gen, device=DEV), n // 20
    keys[at[:k]] = keys[at[k:2 * k]]  # ties
    return keys, torch.arange(n, device=DEV, dtype=torch.int32)


# ---------------------------------------------------------------- what a program keeps

def _flags(case, fused):
    return ((L.GS_FUSED_L1 if fused else 0) | (L.GS_SPLAT_BWD if case["splat"] else 0)
            | (L.GS_RADIX_BIN | L.GS_PERSISTENT if case["radix"] else 0))


def _ordered(case, g, *more):
    """The pool in its spatial order, as the mapping loop keeps it."""
    if not case["ordered"]:
        return (g, *more)
    perm = gsr.spatial_order(g.means)
    return tuple(gsr.permute(x, perm) for x in (g, *more))


def prepare(case, seed):
    kind, deg = case["kind"], case["deg"]
    if kind == "sort":
        return {"case": case, "in": _sort_inputs(case, seed)}
    if kind == "densify":
        p, m, v, accum, denom, normals = _densify_inputs(case, seed)
        return {"case": case, "g": [gsr.Gaussians(*x, deg) for x in (p, m, v)], "stats": (accum, denom, normals)}
    d = _inputs(case, seed)
    if kind in ("autograd", "render"):
        return {"case": case, "d": d, "leaves": [x.requires_grad_(kind == "autograd") for x in d["params"]]}
    tile, wh = _tile(case), d["wh"]
    g = gsr.Gaussians(*d["params"], deg)
    if kind == "pose":
        g, = _ordered(case, g)
        cap = int(gsr.required_pairs(*g.tensors(), d["cams"], wh, deg, tile) * 1.3) + 4096
        plan = gsr.Plan(g.n, deg, wh, tile=tile, lds_batch=64, chunk=1, flags=_flags(case, False), pair_capacity=cap)
        it = gsr.Iteration(plan, g, d["cams"], dL_dcolor=d["gc"], dL_ddepth=d["gd"], pose_grad=True)
        return {"case": case, "it": it, "keep": d}
    g, m, v = _ordered(case, g, gsr.Gaussians(*d["m"], deg), gsr.Gaussians(*d["v"], deg))
    step = torch.full((1,), STEP, dtype=torch.int32, device=DEV)
    cap = int(gsr.required_pairs(*g.tensors(), d["cams"], wh, deg, tile) * 1.3) + 4096
    side = torch.cuda.Stream()
    if kind == "schedule":
        B, (w, h) = case["batch"], wh[0]
        pool = gsr.KeyframePool(d["cams"], d["rgb"].view(len(wh), -1), d["dep"].view(len(wh), -1), B)
        plan = gsr.Plan(g.n, deg, [(w, h)] * B, tile=tile, lds_batch=64, chunk=1, flags=_flags(case, True),
                        pair_capacity=cap)
        it = gsr.Iteration(plan, g, torch.zeros(B, 20, device=DEV), target_rgb=torch.zeros(3 * B * w * h, device=DEV),
                           target_depth=torch.zeros(B * w * h, device=DEV), adam_lrs=LRS, gather=pool,
                           adam_state=(m, v, step))
        ks = gsr.KeyframeScheduler(capacity=64, r0=8, d=4)
        for _ in wh:
            ks.add_keyframe()
        state = {"case": case, "it": it, "pool": pool, "ks": ks, "rng": random.Random(seed + 3), "keep": d}
    else:
        plan = gsr.Plan(g.n, deg, wh, tile=tile, lds_batch=64, chunk=1, flags=_flags(case, not case["ssim"]),
                        pair_capacity=cap)
        it = gsr.Iteration(plan, g, d["cams"], target_rgb=d["rgb"], target_depth=d["dep"] if case["depth"] else None,
                           adam_lrs=LRS, lambda_o=LAMBDA_O if case["reg"] else 0.0,
                           lambda_ssim=LAMBDA_SSIM if case["ssim"] else 0.0, adam_state=(m, v, step))
        state = {"case": case, "it": it, "keep": d}
    torch.cuda.current_stream().synchronize()
    it.capture(side)
    state["side"] = side
    return state


# ---------------------------------------------------------------- one pass

def _frame(it):
    return {"color": it.frame.color, "depth": it.frame.depth, "T": it.frame.T_final, "last": it.frame.last}


def _trained(it):
    return {**_frame(it), "loss": it.frame.loss, "grads": it.grads.tensors(), "params": it.g.tensors(),
            "m": it.m.tensors(), "v": it.v.tensors(), "step": it.step_dev}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "map":
        it = state["it"]
        it.replay()
        return _trained(it)
    if kind == "pose":
        it = state["it"]
        it.enqueue()
        return {**_frame(it), "grads": it.grads.tensors(), "pose": it.dL_dpose}
    if kind == "schedule":
        it, ks = state["it"], state["ks"]
        ids = ks.select_batch([state["rng"].random() for _ in range(case["batch"])])
        state["pool"].select(ids)
        it.replay()
        losses = it.frame.loss.tolist()
        for i, x in zip(ids, losses):
            ks.report(i, x)
        return {**_trained(it), "ids": list(ids)}
    if kind in ("autograd", "render"):
        d, leaves = state["d"], state["leaves"]
        if kind == "render":
            with torch.no_grad():
                color, depth, T = gsr.rasterize(*leaves, d["cams"], d["wh"], case["deg"], tile=_tile(case))
            return {"color": color, "depth": depth, "T": T}
        color, depth, T = gsr.rasterize(*leaves, d["cams"], d["wh"], case["deg"], tile=_tile(case))
        grads = torch.autograd.grad((color, depth), leaves, (d["gc"], d["gd"]))
        return {"color": color, "depth": depth, "T": T, "grads": list(grads)}
    if kind == "densify":
        g, m, v = state["g"]
        accum, denom, normals = state["stats"]
        new = gsr.densify_prune(g, m, v, accum, denom, normals, extent=6.0)
        perm = gsr.spatial_order(new[0].means)
        return {"perm": perm, "pool": [x for y in new for x in gsr.permute(y, perm).tensors()]}
    keys, vals = (x.clone() for x in state["in"])  # the sort works in place
    gsr.sort_pairs(keys, vals, case["bits"])
    return {"keys": keys, "vals": vals}


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    """Each input read once, each output written once, from the case's sizes
    alone.  flops: the alpha evaluations of a surface seen about 10 splats
    deep at every pixel (15 each, 62 with the backward)."""
    kind, n = case["kind"], case["n"]
    if kind == "sort":
        return {"bytes": 24 * n, "flops": 0}
    per = 4 * (11 + 3 * (case["deg"] + 1) ** 2)  # bytes of a Gaussian
    if kind == "densify":
        return {"bytes": 2 * 3 * per * n + 32 * n, "flops": 0}
    sizes = [w * h for _, w, h in _views(case)]
    if kind == "schedule":
        sizes = sizes[: case["batch"]]
    px = sum(sizes)
    if kind == "render":
        return {"bytes": per * n + 20 * px, "flops": 10 * 27 * px}
    if kind in ("autograd", "pose"):  # images and their gradients, parameters, gradients
        return {"bytes": 2 * per * n + (20 + 16) * px, "flops": 10 * (27 + 62) * px}
    # targets in; images and last positions out; parameters and moments in and out, gradients out
    return {"bytes": 7 * per * n + (24 + 12 + 4 * case["depth"]) * px, "flops": 10 * (27 + 62) * px}


# ---------------------------------------------------------------- the same in 64 bits, plain torch

def _project(p, cam, w, h, deg, xi=None):
    """Camera-space quantities of the Gaussians `p` (float64 leaves) in one
    view: mean [n,2], conic [n,3], opacity, colour [n,3], depth, covariance."""
    means, ls, q, logit, sh = p
    c = cam.double()
    fx, fy, cx, cy = c[0], c[1], c[2], c[3]
    R, t = c[4:13].view(3, 3), c[13:16]
    if xi is not None:  # R' = Exp(phi) R, t' = Exp(phi) t + rho, to first order at zero
        z = torch.zeros((), dtype=torch.float64, device=DEV)
        K = torch.stack([z, -xi[5], xi[4], xi[5], z, -xi[3], -xi[4], xi[3], z]).view(3, 3)
        E = torch.eye(3, dtype=torch.float64, device=DEV) + K
        R, t = E @ R, E @ t + xi[:3]
    x = means @ R.T + t
    tz = x[:, 2]
    a, b = x[:, 0] / tz, x[:, 1] / tz
    mx, my = fx * a + cx, fy * b + cy
    lx, ly = 1.3 * w / (2 * fx), 1.3 * h / (2 * fy)
    u, s = torch.minimum(torch.maximum(a, -lx), lx), torch.minimum(torch.maximum(b, -ly), ly)
    r0 = (fx / tz)[:, None] * (R[0] - u[:, None] * R[2])
    r1 = (fy / tz)[:, None] * (R[1] - s[:, None] * R[2])
    qw, qx, qy, qz = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    Q = torch.stack([1 - 2 * (qy * qy + qz * qz), 2 * (qx * qy - qw * qz), 2 * (qx * qz + qw * qy),
                     2 * (qx * qy + qw * qz), 1 - 2 * (qx * qx + qz * qz), 2 * (qy * qz - qw * qx),
                     2 * (qx * qz - qw * qy), 2 * (qy * qz + qw * qx), 1 - 2 * (qx * qx + qy * qy)], 1).view(-1, 3, 3)
    A = torch.exp(ls)[:, None, :] * Q  # Sigma = A A^T
    v0, v1 = (A * r0[:, :, None]).sum(1), (A * r1[:, :, None]).sum(1)
    ca, cb, cc = (v0 * v0).sum(1) + 0.3, (v0 * v1).sum(1), (v1 * v1).sum(1) + 0.3
    det = ca * cc - cb * cb
    conic = torch.stack([cc / det, -cb / det, ca / det], 1)
    o = torch.sigmoid(logit)
    d = means + t @ R  # mean - camera centre, the centre being -R^T t
    d = d / d.norm(dim=1, keepdim=True)
    X, Y, Z = d.unbind(1)
    xx, yy, zz = X * X, Y * Y, Z * Z
    pi = math.pi
    B = [torch.full_like(X, 0.5 / math.sqrt(pi))]
    if deg > 0:
        k = math.sqrt(3 / (4 * pi))
        B += [-k * Y, k * Z, -k * X]
    if deg > 1:
        k = math.sqrt(15 / (4 * pi))
        B += [k * X * Y, -k * Y * Z, math.sqrt(5 / (16 * pi)) * (2 * zz - xx - yy), -k * X * Z, 0.5 * k * (xx - yy)]
    if deg > 2:
        k3, k1 = math.sqrt(35 / (32 * pi)), math.sqrt(21 / (32 * pi))
        B += [-k3 * Y * (3 * xx - yy), math.sqrt(105 / (4 * pi)) * X * Y * Z, -k1 * Y * (4 * zz - xx - yy),
              math.sqrt(7 / (16 * pi)) * Z * (2 * zz - 3 * xx - 3 * yy), -k1 * X * (4 * zz - xx - yy),
              math.sqrt(105 / (16 * pi)) * Z * (xx - yy), -k3 * X * (xx - 3 * yy)]
    raw = (torch.stack(B, 1)[:, :, None] * sh.view(len(X), -1, 3)).sum(1) + 0.5
    return torch.stack([mx, my], 1), conic, o, raw.clamp(min=0), tz, (ca, cc, det)


def _seen(p, cam, w, h, deg):
    """Indices of the Gaussians that reach the view, and their tile boxes (8x8)."""
    near = cam.double()[16]
    got, boxes = [], []
    n = p[0].shape[0]
    for at in range(0, n, 500_000):
        q = [x[at:at + 500_000] for x in p[:4]] + [p[4][at:at + 500_000, :1]]
        m, _, o, _, tz, (ca, cc, det) = _project(q, cam, w, h, 0)
        k = torch.sqrt(2 * torch.log((255 * o).clamp(min=1.0)))
        hx, hy = k * torch.sqrt(ca) + 0.01, k * torch.sqrt(cc) + 0.01
        nx, ny = (w + 7) // 8, (h + 7) // 8
        box = torch.stack([torch.floor((m[:, 0] - hx) / 8).clamp(0, nx), torch.floor((m[:, 1] - hy) / 8).clamp(0, ny),
                           (torch.floor((m[:, 0] + hx) / 8) + 1).clamp(0, nx),
                           (torch.floor((m[:, 1] + hy) / 8) + 1).clamp(0, ny)], 1)
        ok = (tz > near) & (det > 0) & (o >= 1 / 255) & (box[:, 2] > box[:, 0]) & (box[:, 3] > box[:, 1])
        got.append(at + ok.nonzero()[:, 0])
        boxes.append(box[ok].long())
    return torch.cat(got), torch.cat(boxes)


def _lists(box, z, w, h):
    """The (tile, splat) pairs of the boxes, each tile's by (float32 depth, index):
    splat of every pair, and start and length of every tile's list."""
    bw = box[:, 2] - box[:, 0]
    per = bw * (box[:, 3] - box[:, 1])
    who = torch.repeat_interleave(torch.arange(len(per), device=DEV), per)
    k = torch.arange(len(who), device=DEV) - (per.cumsum(0) - per)[who]
    nx, ny = (w + 7) // 8, (h + 7) // 8
    tile = (box[who, 1] + k // bw[who]) * nx + box[who, 0] + k % bw[who]
    order = torch.argsort(z.float()[who], stable=True)
    order = order[torch.argsort(tile[order], stable=True)]
    counts = torch.bincount(tile, minlength=nx * ny)
    return who[order], counts.cumsum(0) - counts, counts


def _blend(m, conic, o, rgb, z, ids, has, tx, ty):
    """Eq. (1) over lists of splats [t, l] at the 64 pixels of each tile:
    colour [t, 64, 3], depth, T and last position."""
    at = ids.reshape(-1)
    take = lambda x: x.index_select(0, at).view(ids.shape + x.shape[1:])
    px = torch.arange(64, device=DEV)
    sx = (tx[:, None] * 8 + (px & 7)).double() + 0.5
    sy = (ty[:, None] * 8 + (px >> 3)).double() + 0.5
    M, C = take(m), take(conic)
    dx, dy = M[:, :, 0, None] - sx[:, None, :], M[:, :, 1, None] - sy[:, None, :]
    power = -0.5 * (C[:, :, 0, None] * dx * dx + C[:, :, 2, None] * dy * dy) - C[:, :, 1, None] * dx * dy
    a = (take(o)[:, :, None] * torch.exp(power)).clamp(max=0.99)
    a = torch.where((a >= 1 / 255) & has[:, :, None], a, torch.zeros_like(a))
    T = torch.cumprod(1 - a, 1)
    blended = (T >= 1e-4).detach()
    front = torch.cat([torch.ones_like(T[:, :1]), T[:, :-1]], 1)
    wgt = torch.where(blended, a * front, torch.zeros_like(a))
    color = torch.einsum("tlp,tlc->tpc", wgt, take(rgb))
    depth = (wgt * take(z)[:, :, None]).sum(1)
    Tf = torch.where(blended, 1 - a, torch.ones_like(a)).prod(1)
    return color, depth, Tf


def _chunks(start, counts):
    """Tiles in groups of like list lengths, at most 2^24 evaluations each."""
    order = torch.argsort(counts)
    host = counts[order].tolist()
    at = next((i for i, c in enumerate(host) if c), len(host))
    while at < len(host):
        to = at + 1
        while to < len(host) and (to - at + 1) * host[to] * 64 <= 1 << 24:
            to += 1
        yield order[at:to], host[to - 1]
        at = to


class _View:
    """One view of a pool in float64: its image, then the gradients of the
    pool for given image gradients."""

    def __init__(self, p, cam, w, h, deg):
        self.p, self.cam, self.w, self.h, self.deg = p, cam, w, h, deg
        with torch.no_grad():
            self.at, box = _seen(p, cam, w, h, deg)
            self.flat = [x.detach() for x in self._shape([x[self.at] for x in p])]
            self.splat, self.start, self.counts = _lists(box, self.flat[4], w, h)
        nx, ny = (w + 7) // 8, (h + 7) // 8
        self.nx = nx
        z = lambda *s: torch.zeros(*s, dtype=torch.float64, device=DEV)
        color, depth, T = z(ny * 8, nx * 8, 3), z(ny * 8, nx * 8), z(ny * 8, nx * 8) + 1
        with torch.no_grad():
            for tiles, longest in _chunks(self.start, self.counts):
                c, d, t = _blend(*self.flat, *self._ids(tiles, longest))
                y, x = self._pixels(tiles)
                color[y, x], depth[y, x], T[y, x] = c, d, t
        bg = cam.double()[17:20]
        self.color = (color + T[:, :, None] * bg)[:h, :w].permute(2, 0, 1).contiguous()
        self.depth, self.T = depth[:h, :w].contiguous(), T[:h, :w].contiguous()

    def _shape(self, q, xi=None):
        return _project(q, self.cam, self.w, self.h, self.deg, xi)[:5]

    def _ids(self, tiles, longest):
        k = torch.arange(longest, device=DEV)
        has = k[None] < self.counts[tiles][:, None]
        at = torch.where(has, self.start[tiles][:, None] + k[None], torch.zeros_like(k)[None])
        return self.splat[at], has, tiles % self.nx, tiles // self.nx

    def _pixels(self, tiles):
        px = torch.arange(64, device=DEV)
        return (tiles // self.nx)[:, None] * 8 + (px >> 3), (tiles % self.nx)[:, None] * 8 + (px & 7)

    def backward(self, gc, gd, into, want_pose=False):
        """Adds the gradients of sum(gc color) + sum(gd depth) to `into` (one
        tensor per parameter); the camera tangent's if wanted."""
        H, W = ((self.h + 7) // 8) * 8, self.nx * 8
        pc, pd = torch.zeros(H, W, 3, dtype=torch.float64, device=DEV), torch.zeros(H, W, dtype=torch.float64, device=DEV)
        pc[:self.h, :self.w] = gc.view(3, self.h, self.w).permute(1, 2, 0)
        pd[:self.h, :self.w] = gd.view(self.h, self.w)
        bg = self.cam.double()[17:20]
        leaf = [x.clone().requires_grad_(True) for x in self.flat]
        for tiles, longest in _chunks(self.start, self.counts):
            c, d, t = _blend(*leaf, *self._ids(tiles, longest))
            y, x = self._pixels(tiles)
            torch.autograd.backward([c + t[:, :, None] * bg, d], [pc[y, x], pd[y, x]])
        q = [x[self.at].clone().requires_grad_(True) for x in self.p]
        xi = torch.zeros(6, dtype=torch.float64, device=DEV, requires_grad=want_pose)
        if leaf[0].grad is not None:
            torch.autograd.backward(list(self._shape(q, xi if want_pose else None)), [x.grad for x in leaf])
            for g, x in zip(into, q):
                g.index_add_(0, self.at, x.grad)
        return xi.grad if want_pose and xi.grad is not None else torch.zeros(6, dtype=torch.float64, device=DEV)


@functools.lru_cache(maxsize=None)
def _window():
    x = np.arange(11) - 5
    g = np.exp(-x * x / (2 * 1.5 ** 2))
    g /= g.sum()
    return torch.tensor(np.outer(g, g), device=DEV).expand(3, 1, 11, 11).contiguous()


def _loss(case, color, depth, rgb, dep):
    l1 = (color - rgb).abs().mean()
    if case["ssim"]:
        blur = lambda x: F.conv2d(x[None], _window(), padding=5, groups=3)[0]
        a, b = blur(color), blur(rgb)
        va, vb, ab = blur(color * color) - a * a, blur(rgb * rgb) - b * b, blur(color * rgb) - a * b
        ssim = ((2 * a * b + 1e-4) * (2 * ab + 9e-4)) / ((a * a + b * b + 1e-4) * (va + vb + 9e-4))
        l1 = (1 - LAMBDA_SSIM) * l1 + LAMBDA_SSIM * (1 - ssim.mean())
    return l1 + LAMBDA_DEPTH * (depth - dep).abs().mean() if case["depth"] else l1


def _cut(x, wh, channels):
    out, at = [], 0
    for w, h in wh:
        out.append(x[at:at + channels * w * h].double().view(*((3, h, w) if channels == 3 else (h, w))))
        at += channels * w * h
    return out


def _order(means):
    """The spatial order: Morton code of the means in their box, stable."""
    lo, hi = means.min(0).values, means.max(0).values
    q = (((means - lo) / (hi - lo)).clamp(0, 1) * 1023.0).long()
    code = torch.zeros_like(q[:, 0])
    for b in range(10):
        for d in range(3):
            code |= ((q[:, d] >> b) & 1) << (3 * b + d)
    return torch.argsort(code, stable=True)


def _exact_densify(case, seed):
    p, m, v, accum, denom, normals = _densify_inputs(case, seed)
    keep = torch.sigmoid(p[3]) >= 0.02
    chosen = (denom > 0) & (accum / denom >= 0.001)
    split = chosen & (torch.exp(p[1].max(1).values) > 0.06)
    count = torch.where(keep, 1 + chosen.int(), 0)
    who = torch.repeat_interleave(torch.arange(case["n"], device=DEV), count)
    child = torch.arange(len(who), device=DEV) - (count.cumsum(0) - count)[who]
    new = [x[who].double() for x in p]
    s = split[who]
    q = new[2] / new[2].norm(dim=1, keepdim=True)
    off = torch.exp(new[1]) * normals[who, child.clamp(max=1)].double()
    uv = torch.linalg.cross(q[:, 1:], off)
    off = off + 2 * (q[:, :1] * uv + torch.linalg.cross(q[:, 1:], uv))
    new[0] = torch.where(s[:, None], new[0] + off, new[0])
    new[1] = torch.where(s[:, None], new[1] - math.log(1.6), new[1])
    fresh = (s | (child > 0))
    moved = [[torch.where(fresh.view(-1, *[1] * (x.dim() - 1)), 0.0, x[who].double()) for x in y] for y in (m, v)]
    perm = _order(new[0].float())
    return {"perm": None, "pool": [x[perm] for y in (new, *moved) for x in y]}


def exact(case, seed):
    kind, deg = case["kind"], case["deg"]
    if kind == "sort":
        return None  # whole numbers
    if kind == "densify":
        return _exact_densify(case, seed)
    d = _inputs(case, seed)
    if kind in ("map", "schedule", "pose") and case["ordered"]:
        perm = _order(d["params"][0])
        for f in ("params", "m", "v"):
            if f in d:
                d[f] = [x[perm] for x in d[f]]
    p = [x.detach().double() for x in d["params"]]
    wh, cams = d["wh"], d["cams"]
    rgb, dep = _cut(d["rgb"], wh, 3), _cut(d["dep"], wh, 1)
    if kind in ("pose", "autograd"):
        gc, gd = _cut(d["gc"], wh, 3), _cut(d["gd"], wh, 1)
    use = range(len(wh))
    if kind == "schedule":  # the first selection: every keyframe still has its turns
        rng, left, use = random.Random(seed + 3), list(use), []
        for _ in range(case["batch"]):
            use.append(left.pop(int(rng.random() * len(left))))
    into = [torch.zeros_like(x) for x in p]
    color, depth, T, losses, pose = [], [], [], [], []
    for i in use:
        view = _View(p, cams[i], *wh[i], deg)
        color.append(view.color.reshape(-1))
        depth.append(view.depth.reshape(-1))
        T.append(view.T.reshape(-1))
        if kind == "render":
            continue
        if kind in ("pose", "autograd"):
            pose.append(view.backward(gc[i], gd[i], into, kind == "pose"))
            continue
        c, z = view.color.clone().requires_grad_(True), view.depth.clone().requires_grad_(True)
        loss = _loss(case, c, z, rgb[i], dep[i])
        g = torch.autograd.grad(loss, (c, z), allow_unused=True)
        losses.append(loss.detach())
        view.backward(g[0], torch.zeros_like(z) if g[1] is None else g[1], into)
    out = {"color": torch.cat(color), "depth": torch.cat(depth), "T": torch.cat(T)}
    if kind == "render":
        return out
    out["grads"] = into
    if kind == "autograd":
        return out
    if kind == "pose":
        return {**out, "last": None, "pose": torch.stack(pose)}
    step, params, ms, vs = STEP + 1, [], [], []
    for f, x, g, m, v in zip(FIELDS, p, into, d["m"], d["v"]):
        if f == "opacity_logits" and case["reg"]:
            o = torch.sigmoid(x)
            g = g + LAMBDA_O / case["n"] * o * (1 - o)
        m, v = BETA1 * m.double() + (1 - BETA1) * g, BETA2 * v.double() + (1 - BETA2) * g * g
        params.append(x - LRS[f] / (1 - BETA1 ** step) * m / (torch.sqrt(v / (1 - BETA2 ** step)) + EPS))
        ms.append(m)
        vs.append(v)
    return {**out, "last": None, "loss": torch.stack(losses), "params": params, "m": ms, "v": vs, "step": None,
            **({"ids": None} if kind == "schedule" else {})}
