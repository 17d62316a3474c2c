"""Performance cases of the per-object NeRF library, each one pass through a
public entry point at a size that the repository's own workloads, tests or
benchmark use, or at a ragged size of the same range.

listed() names the cases, draw() gives further ones of the same ranges,
prepare() builds what a user's program holds before the call (inputs from the
seed alone, on the GPU), run() is the timed pass, work() the bytes and
operations the pass cannot do without, and exact() the same outputs from
plain torch in FP64.

Inputs: cameras on a sphere of radius 1.5 around the object look at its unit
box; the targets are a closed-form shaded sphere; the prior is a blurred
sphere occupancy; the networks hold weights of the size training gives them
(table entries up to 0.5, Xavier layers, a density row that spreads
sigma over two decades), and the optimiser's moments are those of a run under
way, so that an update is a smooth function of the gradient.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch
import torch.nn.functional as F

from paper_2503_01582_amd import api, autograd, autotune, batch, meta, trainer
from synth.arch import Arch
from synth.workloads import LossSpec, SampleSpec

DEV = "cuda"
NEAR, FAR = 0.5, 2.5
F64 = torch.float64


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # the sampler of one mapping iteration at the paper's settings (4096 rays, 32 coarse bins, 32 draws):
        # the smallest call of the library
        dict(name="sample_4096", kind="sample", rays=4096, coarse=32, fine=32, merge=False, prior_res=64),
        # canonical yaw of an object seen from a few viewpoints (a depth cloud, one yaw per degree)
        dict(name="yaw_8927x360", kind="yaw", points=8927, yaws=360, prior_res=64),
        # the prior refreshed from the object's network every 50 iterations
        dict(name="prior_refresh_64", kind="refresh", res=64, levels=16, log2_table=19, width=64, hidden=2,
             mlp="fp32", table="fp32"),
        # a view rendered without loss or gradient, odd numbers of pixels and samples
        dict(name="view_307x211", kind="view", width_px=307, height_px=211, fine=33, levels=12, log2_table=15,
             width=32, hidden=1, mlp="fp32", table="fp32"),
        # one training iteration of one object at the paper's ray count (launches and latency count)
        dict(name="step_small", kind="step", rays=4096, coarse=0, fine=32, merge=False, prior_res=0, levels=8,
             log2_table=14, width=64, hidden=1, mlp="fp32", table="fp32", lambda_d=0.0, lambda_sigma=0.0),
        # one training iteration with prior-based sampling and large tables
        dict(name="step_prior", kind="step", rays=65536, coarse=16, fine=48, merge=True, prior_res=64, levels=16,
             log2_table=19, width=64, hidden=2, mlp="fp32", table="fp32", lambda_d=0.0, lambda_sigma=0.0),
        # the renderer under torch.autograd with a loss of colour and depth, forward and backward, ragged
        dict(name="autograd_30011", kind="autograd", rays=30011, coarse=16, fine=48, prior_res=48, recompute=False,
             levels=12, log2_table=17, width=64, hidden=2, mlp="fp32", table="fp32"),
        # the same in the form that keeps no activations, the widest network in 16 bits, several passes
        dict(name="autograd_recompute_fp16", kind="autograd", rays=70001, coarse=16, fine=40, prior_res=64,
             recompute=True, levels=16, log2_table=18, width=128, hidden=2, mlp="fp16", table="fp16"),
        # a map's many small objects trained side by side, one eager iteration of all
        dict(name="batch16_small", kind="batch", objects=16, rays=18000, objects_seed=3, mlp="fp32", table="fp32",
             graph=False),
        # 24 objects of every size and architecture in FP32
        dict(name="batch24_fp32", kind="batch", objects=24, rays=338571, objects_seed=4, mlp="fp32", table="fp32",
             graph=False),
        # 48 objects in reduced precision with loss scaling, the step replayed from a graph: the largest
        dict(name="batch48_bf16", kind="batch", objects=48, rays=1 << 20, objects_seed=5, mlp="bf16", table="fp16",
             graph=True),
        # a meta-learning iteration: 8 tasks, 2 inner steps, the outer update
        dict(name="reptile_8x4096", kind="reptile", tasks=8, rays=4096, fine=32, inner_steps=2, levels=12,
             log2_table=17, width=64, hidden=2, mlp="fp32", table="fp32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_net(rng):
    mlp = rng.choice(["fp32", "fp32", "bf16", "fp16"])
    return dict(levels=rng.choice([8, 12, 16]), log2_table=rng.randint(14, 19), width=rng.choice([32, 64, 128]),
                hidden=rng.choice([1, 2]), mlp=mlp, table="fp32" if mlp == "fp32" else rng.choice(["fp32", "fp16"]))


def draw(rng: random.Random):
    kind = rng.choice(["sample", "yaw", "refresh", "view", "step", "step", "autograd", "autograd", "batch", "batch",
                       "reptile"])
    if kind == "sample":
        return dict(kind=kind, rays=_log(rng, 1000, 1 << 18), coarse=rng.choice([16, 24, 32]),
                    fine=rng.randint(16, 64), merge=rng.random() < 0.5, prior_res=rng.randint(32, 64))
    if kind == "yaw":
        return dict(kind=kind, points=_log(rng, 500, 60000), yaws=rng.choice([72, 180, 360, 720]),
                    prior_res=rng.randint(32, 64))
    if kind == "refresh":
        return dict(kind=kind, res=rng.randint(32, 96), **_draw_net(rng))
    if kind == "view":
        return dict(kind=kind, width_px=_log(rng, 48, 640), height_px=_log(rng, 48, 480), fine=rng.randint(16, 64),
                    **_draw_net(rng))
    if kind == "step":
        merge = rng.random() < 0.5
        return dict(kind=kind, rays=_log(rng, 1024, 1 << 17), coarse=16, fine=rng.randint(24, 48), merge=merge,
                    prior_res=rng.randint(32, 64), lambda_d=rng.choice([0.0, 0.1]),
                    lambda_sigma=rng.choice([0.0, 0.01]), **_draw_net(rng))
    if kind == "autograd":
        return dict(kind=kind, rays=_log(rng, 1024, 1 << 17), coarse=16, fine=rng.randint(24, 48),
                    prior_res=rng.randint(32, 64), recompute=rng.random() < 0.4, **_draw_net(rng))
    if kind == "batch":
        n = rng.randint(3, 32)
        mlp = rng.choice(["fp32", "bf16", "fp16"])
        return dict(kind=kind, objects=n, rays=n * _log(rng, 500, 12000) + rng.randint(0, 63),
                    objects_seed=rng.randint(10, 10 ** 6), mlp=mlp, table="fp32" if mlp == "fp32" else "fp16",
                    graph=rng.random() < 0.5)
    net = dict(_draw_net(rng), mlp="fp32", table="fp32", log2_table=rng.randint(14, 17), width=rng.choice([32, 64]))
    return dict(kind=kind, tasks=rng.randint(2, 8), rays=_log(rng, 1000, 8192), fine=rng.randint(16, 48),
                inner_steps=rng.randint(1, 3), **net)


# ------------------------------------------------------------------ inputs

def _gen(*seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(np.random.SeedSequence(seed).generate_state(1, np.uint64)[0] >> np.uint64(1)))
    return g


def _uniform(g, shape, lo, hi):
    return torch.rand(shape, generator=g, device=DEV) * (hi - lo) + lo


def _arch(c):
    return Arch(n_levels=c["levels"], log2_table=c["log2_table"], width=c["width"], hidden=c["hidden"],
                mlp_dtype=c["mlp"], table_dtype=c["table"])


def _params(arch, g):
    """Weights of a network under training."""
    parts = [_uniform(g, (arch.n_table_params,), -0.5, 0.5)]
    for k, (o, i) in enumerate(arch.layer_shapes()):
        w = _uniform(g, (o, i), -1.0, 1.0) * math.sqrt(6.0 / (o + i))
        if k == arch.hidden:
            w[0] *= 4.0
        parts.append(w.reshape(-1))
    return torch.cat(parts)


def _prior(res, g):
    """[R, R, R] blurred sphere occupancy plus a floor, x fastest."""
    c = 0.5 + _uniform(g, (3,), -0.04, 0.04)
    a = torch.arange(res, device=DEV, dtype=torch.float32) / (res - 1)
    r = ((a[:, None, None] - c[2]) ** 2 + (a[None, :, None] - c[1]) ** 2 + (a[None, None, :] - c[0]) ** 2).sqrt()
    return (torch.sigmoid((0.3 - r) / 0.04) + 0.01).contiguous()


def _pose(rng):
    """Row-major 3x4 world -> unit box, and the object's rotation and shift."""
    th = rng.uniform(0.0, 2.0 * math.pi)
    rot = np.array([[math.cos(th), -math.sin(th), 0.0], [math.sin(th), math.cos(th), 0.0], [0.0, 0.0, 1.0]])
    shift = np.array([rng.uniform(-2, 2), rng.uniform(-2, 2), rng.uniform(-0.2, 0.2)])
    A = np.empty((3, 4))
    A[:, :3] = rot.T
    A[:, 3] = 0.5 - rot.T @ shift
    return A.astype(np.float32), rot, shift


def _normalise(v):
    return v / v.norm(dim=-1, keepdim=True)


def _targets(o, d):
    """Colour, depth and mask of a shaded sphere of radius 0.3 (object frame, centre 0)."""
    b = (o * d).sum(1)
    disc = b * b - (o * o).sum(1) + 0.09
    hit = disc > 0
    depth = torch.where(hit, -b - disc.clamp_min(0).sqrt(), torch.zeros_like(b))
    n = (o + depth[:, None] * d) / 0.3
    rgb = torch.where(hit[:, None], 0.5 + 0.35 * n, torch.zeros_like(n))
    return rgb.float().contiguous(), depth.float().contiguous(), hit.to(torch.uint8)


def _rays(n, fine, pose, g):
    """n rays of 16 cameras on the sphere towards points of the object's box."""
    _, rot, shift = pose
    cams = 1.5 * _normalise(torch.randn((16, 3), generator=g, device=DEV, dtype=F64))
    o = cams[torch.randint(0, 16, (n,), generator=g, device=DEV)]
    tgt = torch.rand((n, 3), generator=g, device=DEV, dtype=F64) * 0.9 - 0.45
    return _world(o, _normalise(tgt - o), fine, rot, shift, g)


def _view(w, h, fine, pose, g):
    """The pixel rays of one camera (60 degrees across), row by row; some miss the box."""
    _, rot, shift = pose
    eye = _normalise(torch.randn(3, generator=g, device=DEV, dtype=F64) * torch.tensor([1.0, 1.0, 0.5], device=DEV))
    right = _normalise(torch.linalg.cross(-eye, torch.tensor([0.0, 0.0, 1.0], device=DEV, dtype=F64)))
    up = torch.linalg.cross(right, -eye)
    f = 0.5 * w / math.tan(math.radians(30.0))
    x = (torch.arange(w, device=DEV, dtype=F64) + 0.5 - 0.5 * w) / f
    y = -(torch.arange(h, device=DEV, dtype=F64) + 0.5 - 0.5 * h) / f
    d = x[None, :, None] * right + y[:, None, None] * up - eye
    d = _normalise(d.reshape(-1, 3))
    return _world((1.5 * eye).expand_as(d), d, fine, rot, shift, g)


def _world(o, d, fine, rot, shift, g):
    rgb, depth, mask = _targets(o, d)
    R = torch.as_tensor(rot, device=DEV)
    u = torch.randint(0, 1 << 24, (o.shape[0], fine), generator=g, device=DEV, dtype=torch.int32)
    return dict(rays_o=(o @ R.T + torch.as_tensor(shift, device=DEV)).float().contiguous(),
                rays_d=(d @ R.T).float().contiguous(), xi=((u.double() + 0.5) * 2.0 ** -24).float(),
                tgt_rgb=rgb, tgt_depth=depth, mask=mask)


def _moments(model, n_rays, g):
    """Adam moments of a run under way: gradients of the order of 0.03 / rays."""
    s = 0.03 / n_rays
    model.adam_m.copy_(torch.randn(model.adam_m.shape, generator=g, device=DEV) * (0.3 * s))
    model.adam_v.copy_((_uniform(g, model.adam_v.shape, 0.5, 1.5) * s) ** 2)


def _spec(c):
    coarse = c.get("coarse", 0)
    return SampleSpec(n_coarse=coarse, n_fine=c["fine"], include_coarse=bool(c.get("merge", coarse > 0)),
                      uniform_only=not c.get("prior_res", 0), near=NEAR, far=FAR)


def _scale(c):
    """Initial loss scale of the 16-bit networks."""
    return None if c["mlp"] == "fp32" else 4096.0


def _inputs(c, seed):
    """Pose, rays, prior and weights of a single-object case."""
    g, rng = _gen(seed, 1), np.random.default_rng([seed, 2])
    pose = _pose(rng)
    if c["kind"] == "view":
        rays = _view(c["width_px"], c["height_px"], c["fine"], pose, g)
    else:
        rays = _rays(c["rays"], c["fine"], pose, g)
    prior = _prior(c["prior_res"], g) if c.get("prior_res", 0) else None
    params = _params(_arch(c), g) if "levels" in c else None
    return pose, rays, prior, params, g


def _objects(c):
    """Architectures and ray counts of a batch (the recipe of the many-object workloads)."""
    rng = random.Random(c["objects_seed"])
    archs, weight = [], []
    for _ in range(c["objects"]):
        archs.append(Arch(n_levels=rng.choice([8, 12, 16]), log2_table=rng.randint(14, 19),
                          width=rng.choice([32, 64, 128]), hidden=rng.choice([1, 2]), mlp_dtype=c["mlp"],
                          table_dtype=c["table"]))
        weight.append(math.exp(rng.uniform(math.log(1024.0), math.log(65536.0))))
    counts = [int(c["rays"] * w / sum(weight)) for w in weight]
    counts[0] += c["rays"] - sum(counts)
    return archs, counts


BATCH_SPEC = SampleSpec(n_coarse=16, n_fine=48, include_coarse=True, uniform_only=False, near=NEAR, far=FAR)
INNER_LR, META_STEP = 20.0, 0.5
ADAM_STEP = 100  # iterations behind the state of the training cases


def _batch_inputs(c, seed):
    archs, counts = _objects(c)
    g, rng = _gen(seed, 1), np.random.default_rng([seed, 2])
    objs, rays, params = [], [], []
    for a, n in zip(archs, counts):
        pose = _pose(rng)
        prior = _prior(int(rng.integers(32, 65)), g)
        rays.append(_rays(n, BATCH_SPEC.n_fine, pose, g))
        params.append(_params(a, g))
        objs.append(batch.BatchObject(a, n, prior, pose[0]))
    return objs, {k: torch.cat([r[k] for r in rays]) for k in rays[0]}, params, g


def _cloud(c, seed):
    """Depth cloud of an elongated box seen from outside, and the prior grid."""
    g = _gen(seed, 1)
    p = _uniform(g, (c["points"], 3), -1.0, 1.0)
    face = torch.randint(0, 3, (c["points"],), generator=g, device=DEV)
    p[torch.arange(c["points"], device=DEV), face] = torch.sign(_uniform(g, (c["points"],), -1.0, 1.0))
    p *= torch.tensor([0.45, 0.25, 0.3], device=DEV)
    return p.contiguous(), _prior(c["prior_res"], g)


# ------------------------------------------------------------------ prepare and run

def prepare(c, seed):
    kind = c["kind"]
    if kind == "yaw":
        pts, prior = _cloud(c, seed)
        return dict(kind=kind, pts=pts, prior=prior, yaws=c["yaws"])
    if kind == "batch":
        return _prepare_batch(c, seed)
    if kind == "reptile":
        return _prepare_reptile(c, seed)
    if kind == "refresh":
        arch = _arch(c)
        return dict(kind=kind, model=api.Model(arch, _params(arch, _gen(seed, 1)), DEV), res=c["res"])
    pose, rays, prior, params, g = _inputs(c, seed)
    spec = _spec(c)
    s = dict(kind=kind, spec=spec, pose=pose[0], rays=rays, prior=prior)
    if kind == "sample":
        return s
    arch = _arch(c)
    if kind == "step":
        loss = LossSpec(0, c["lambda_d"], c["lambda_sigma"])
        tr = trainer.Trainer(arch, params, spec, loss, device=DEV, loss_scale=_scale(c))
        _moments(tr.model, c["rays"], g)
        tr.model.step = ADAM_STEP
        b = trainer.DeviceBatch(world_to_obj=pose[0], prior=prior, bg=None, **rays)
        return dict(s, trainer=tr, batch=b)
    s["model"] = api.Model(arch, params, DEV, loss_scale=_scale(c))
    if kind == "view":
        s["ws"] = api.Workspace(DEV)
    else:
        s["model"].params.requires_grad_(True)
        s["recompute"] = c["recompute"]
    return s


def _prepare_batch(c, seed):
    objs, rays, params, g = _batch_inputs(c, seed)
    tr = batch.BatchTrainer(objs, params, BATCH_SPEC, LossSpec(), device=DEV, loss_scale=_scale(c),
                            tiles=autotune.tiles_for([o.arch for o in objs]))
    for k, v in rays.items():
        getattr(tr, k).copy_(v)
    _moments(tr.model, c["rays"] / c["objects"], g)
    tr.model.step.fill_(ADAM_STEP)
    if c["graph"]:
        tr.capture()
    return dict(kind="batch", trainer=tr, graph=c["graph"])


def _prepare_reptile(c, seed):
    g, rng = _gen(seed, 1), np.random.default_rng([seed, 2])
    arch, pose = _arch(c), _pose(rng)
    tr = meta.ReptileTrainer(arch, _params(arch, g), c["tasks"], c["rays"], _spec(c), LossSpec(), inner_lr=INNER_LR,
                             beta=META_STEP, world_to_obj=pose[0], device=DEV)
    rays = [_rays(c["rays"], c["fine"], pose, g) for _ in range(c["tasks"])]
    return dict(kind="reptile", trainer=tr, steps=c["inner_steps"],
                rays={k: torch.cat([r[k] for r in rays]) for k in rays[0]})


def run(s):
    kind = s["kind"]
    if kind == "yaw":
        return api.prenom_canonical_yaw(s["pts"], s["prior"], s["yaws"])
    if kind == "refresh":
        return api.prenom_prior_refresh(s["model"], s["res"])
    if kind == "step":
        tr = s["trainer"]
        out = tr.step(s["batch"])
        return dict(out, params=tr.model.params, adam_m=tr.model.adam_m)
    if kind == "batch":
        tr = s["trainer"]
        out = tr.replay() if s["graph"] else tr.step()
        return dict(out, params=tr.model.params, adam_m=tr.model.adam_m)
    if kind == "reptile":
        tr = s["trainer"]
        tr.load_rays(**s["rays"])
        for _ in range(s["steps"]):
            out = tr.step()
        tr.outer()
        return dict(out, theta=tr.theta)
    r = s["rays"]
    samp = api.prenom_sample(s["spec"], r["rays_o"], r["rays_d"], r["xi"], s["pose"], s["prior"])
    if kind == "sample":
        return dict(ray_obj=samp.ray_obj, t=samp.t, dt=samp.dt, bins=samp.bins, flags=samp.flags)
    model = s["model"]
    if kind == "view":
        ws = s["ws"].get(model.arch, samp.t.shape[0], samp.n_samples)
        out = api.prenom_render_fwd(model, samp, None, ws, want_loss=False)
        return dict(rgb=out["rgb"], depth=out["depth"], opacity=out["opacity"])
    rgb, depth, opacity = autograd.render(model, samp, None, s["recompute"])
    m = r["mask"].float()
    loss = ((rgb - r["tgt_rgb"]) ** 2).mean() + 0.1 * (m * (depth - r["tgt_depth"]) ** 2).mean()
    model.params.grad = None
    loss.backward()
    return dict(rgb=rgb.detach(), depth=depth.detach(), opacity=opacity.detach(), loss=loss.detach(),
                grad=model.params.grad)


# ------------------------------------------------------------------ work

def _net_flops(arch):
    """Per point: the trilinear blend of every level and the network's products."""
    return arch.n_levels * 8 * 2 * arch.n_features + 2 * arch.n_mlp_params


def work(c):
    kind = c["kind"]
    if kind == "yaw":
        return dict(bytes=12.0 * c["points"] + 4.0 * c["prior_res"] ** 3 + 56.0 * c["yaws"],
                    flops=71.0 * c["points"] * c["yaws"])
    if kind == "refresh":
        a, n = _arch(c), c["res"] ** 3
        return dict(bytes=4.0 * n + (2.0 if c["table"] == "fp16" else 4.0) * a.n_params, flops=float(n) * _net_flops(a))
    if kind == "batch":
        archs, counts = _objects(c)
        S, nf = BATCH_SPEC.n_samples, BATCH_SPEC.n_fine
        return dict(bytes=sum(n * (24.0 + 4 * nf + 17 + 20) + 24.0 * a.n_params for a, n in zip(archs, counts)),
                    flops=sum(3.0 * n * S * _net_flops(a) for a, n in zip(archs, counts)))
    rays = c["width_px"] * c["height_px"] if kind == "view" else c["rays"]
    S = _spec(c).n_samples
    per_ray = 24.0 + 4 * c["fine"]
    if kind == "sample":
        return dict(bytes=rays * (per_ray + 24 + 8 * S + 4 * c["fine"] + 1) + 4.0 * c["prior_res"] ** 3,
                    flops=rays * (100.0 * c["coarse"] + 20.0 * c["fine"]))
    a = _arch(c)
    if kind == "view":
        return dict(bytes=rays * (per_ray + 20) + 4.0 * a.n_params, flops=float(rays) * S * _net_flops(a))
    if kind == "step":
        return dict(bytes=rays * (per_ray + 17 + 20) + 24.0 * a.n_params, flops=3.0 * rays * S * _net_flops(a))
    if kind == "autograd":
        return dict(bytes=rays * (per_ray + 17 + 20) + 8.0 * a.n_params, flops=3.0 * rays * S * _net_flops(a))
    q, B = c["inner_steps"], c["tasks"]
    return dict(bytes=B * rays * (per_ray + 17 + 20) + 8.0 * a.n_params * (1 + B * q),
                flops=3.0 * q * B * rays * S * _net_flops(a))


# ------------------------------------------------------------------ the same in FP64

CHUNK = 1 << 19          # samples held at once
MOST_GRAD = 1 << 25      # samples whose gradient is computed here
MOST_FWD = 3 << 25       # samples whose forward is computed here


def _lookup(grid, x):
    """Trilinear, vertex-aligned lookup of grid [R, R, R] (x fastest) at x [..., 3]."""
    R = grid.shape[0]
    g = x.nan_to_num(0.0).clamp(0.0, 1.0) * (R - 1)
    i = g.floor().clamp_max(R - 2)
    f = g - i
    i = i.long()
    flat, s = grid.double().reshape(-1), 0.0
    for cz in (0, 1):
        for cy in (0, 1):
            for cx in (0, 1):
                w = 1.0
                for a, ca in enumerate((cx, cy, cz)):
                    w = w * (f[..., a] if ca else 1.0 - f[..., a])
                s = s + w * flat[(i[..., 0] + cx) + R * ((i[..., 1] + cy) + R * (i[..., 2] + cz))]
    return s


def _sample64(spec, rays, pose, prior):
    A = torch.as_tensor(pose, device=DEV).double().reshape(3, 4)
    o = rays["rays_o"].double() @ A[:, :3].T + A[:, 3]
    d = rays["rays_d"].double() @ A[:, :3].T
    inf = torch.full_like(o, math.inf)
    ta, tb, flat = -o / d, (1.0 - o) / d, d == 0
    enter = torch.where(flat, -inf, torch.minimum(ta, tb)).amax(1)
    leave = torch.where(flat, inf, torch.maximum(ta, tb)).amin(1)
    tn, tf = enter.clamp_min(spec.near), leave.clamp_max(spec.far)
    hit = (tn < tf) & ~(flat & ((o < 0) | (o > 1))).any(1)
    span, length = tf - tn, d.norm(dim=1)
    u = (torch.arange(spec.n_fine, device=DEV) + rays["xi"].double()) / spec.n_fine
    t = tn[:, None] + u * span[:, None]
    if spec.n_coarse:
        delta = span / spec.n_coarse
        mid = tn[:, None] + (torch.arange(spec.n_coarse, device=DEV) + 0.5) * delta[:, None]
        if prior is not None and not spec.uniform_only:
            sig = _lookup(prior, o[:, None] + mid[..., None] * d[:, None])
            sp = torch.cumsum(sig * (delta * length)[:, None], 1)
            cdf = torch.expm1(-sp) / torch.expm1(-sp[:, -1:])
            cdf = torch.cat([torch.zeros_like(sp[:, :1]), cdf[:, :-1], torch.ones_like(sp[:, :1])], 1)
            b = torch.searchsorted(cdf[:, 1:].contiguous(), u).clamp_max(spec.n_coarse - 1)
            lo, hi = cdf.gather(1, b), cdf.gather(1, b + 1)
            drawn = tn[:, None] + delta[:, None] * (b + (u - lo) / (hi - lo))
            t = torch.where((-torch.expm1(-sp[:, -1:]) < spec.eps), t, drawn)
        if spec.include_coarse:
            t = torch.sort(torch.cat([mid, t], 1), 1).values
    dt = torch.cat([t[:, 1:], tf[:, None]], 1).sub(t) * length[:, None]
    t, dt = (torch.where(hit[:, None], v, torch.zeros_like(v)) for v in (t, dt))
    return torch.cat([o, d], 1), t, dt, hit


def _features(arch, tables, x):
    """Hash encoding of FP32 positions x [n, 3] (as FP64 values): [n, L F]."""
    T, out = arch.table_size, []
    for l, N in enumerate(arch.resolutions):
        xs = x * N
        c = xs.floor().clamp(0, N - 1)
        f = xs - c
        c = c.long()
        dense, acc = (N + 1) ** 3 <= T, 0.0
        for e in range(8):
            v = [c[:, a] + (e >> a & 1) for a in range(3)]
            if dense:
                row = v[0] + (N + 1) * (v[1] + (N + 1) * v[2])
            else:
                row = (v[0] ^ (v[1] * 2654435761 & 0xFFFFFFFF) ^ (v[2] * 805459861 & 0xFFFFFFFF)) & (T - 1)
            w = 1.0
            for a in range(3):
                w = w * (f[:, a] if e >> a & 1 else 1.0 - f[:, a])
            acc = acc + w[:, None] * torch.index_select(tables[l], 0, row)
        out.append(acc)
    return torch.cat(out, 1)


def _split(arch, p):
    tables = p[:arch.n_table_params].reshape(arch.n_levels, arch.table_size, arch.n_features)
    layers, at = [], arch.n_table_params
    for o, i in arch.layer_shapes():
        layers.append(p[at:at + o * i].reshape(o, i))
        at += o * i
    return tables, layers


def _net(arch, p, x):
    tables, layers = _split(arch, p)
    h = _features(arch, tables, x)
    for w in layers[:-1]:
        h = F.relu(h @ w.T)
    o = h @ layers[-1].T
    return torch.exp(o[:, 0]), torch.sigmoid(o[:, 1:])


def _positions(ray_obj, t):
    """clamp(fma(t, d, o)) rounded to FP32 once, as FP64 values."""
    o, d = ray_obj[:, None, :3].float().double(), ray_obj[:, None, 3:].float().double()
    return (o + t.float().double()[..., None] * d).float().clamp(0.0, 1.0).double()


def _render64(arch, p, samp, loss_of=None, grad=False):
    """rgb, depth, opacity and the summed loss of the sampled rays; loss_of(rows,
    rgb, depth, sigma) is a part's loss.  With grad, also its gradient."""
    ray_obj, t, dt, hit = samp
    n, S = t.shape
    p = p.detach().double().requires_grad_(grad)
    rgb, depth, opacity, total = [], [], [], torch.zeros((), dtype=F64, device=DEV)
    step = max(1, CHUNK // S)
    with torch.set_grad_enabled(grad):
        for r0 in range(0, n, step):
            rows = slice(r0, min(n, r0 + step))
            x = _positions(ray_obj[rows], t[rows])
            k = x.shape[0]
            sigma, col = _net(arch, p, x.reshape(-1, 3))
            sigma, col = sigma.reshape(k, S), col.reshape(k, S, 3)
            live = hit[rows].double()
            tau = sigma * dt[rows].float().double() * live[:, None]
            acc = torch.cumsum(tau, 1)
            w = torch.exp(-(acc - tau)) * -torch.expm1(-tau)
            C, D, O = (w[..., None] * col).sum(1), (w * t[rows].float().double()).sum(1), w.sum(1)
            if loss_of is not None:
                part = loss_of(rows, C, D, sigma * live[:, None])
                total = total + part.detach()
                if grad:
                    part.backward()
            rgb.append(C.detach())
            depth.append(D.detach())
            opacity.append(O.detach())
    out = dict(rgb=torch.cat(rgb), depth=torch.cat(depth), opacity=torch.cat(opacity), loss=total)
    return (out, p.grad) if grad else (out, None)


def _mse_loss(rays, n, lambda_d, lambda_sigma):
    def part(rows, C, D, sigma):
        m = rays["mask"][rows].double()
        loss = ((C - rays["tgt_rgb"][rows].double()) ** 2).sum() / (3 * n)
        if lambda_d:
            loss = loss + lambda_d * (m * (D - rays["tgt_depth"][rows].double()) ** 2).sum() / n
        if lambda_sigma:
            loss = loss + lambda_sigma * ((1 - m)[:, None] * sigma).sum() / n
        return loss
    return part


def _adam64(p, g, m, v, step=ADAM_STEP + 1, lr=1e-2, b1=0.9, b2=0.99, eps=1e-15):
    b1, b2, lr, eps = (float(np.float32(x)) for x in (b1, b2, lr, eps))
    m = b1 * m.double() + (1 - b1) * g
    v = b2 * v.double() + (1 - b2) * g * g
    return p.double() - lr * (m / (1 - b1 ** step)) / ((v / (1 - b2 ** step)).sqrt() + eps), m


class _Moments:
    def __init__(self, n):
        self.adam_m = torch.empty(n, device=DEV)
        self.adam_v = torch.empty(n, device=DEV)


def exact(c, seed):
    kind = c["kind"]
    if kind == "yaw":
        return _exact_yaw(c, seed)
    if kind == "refresh":
        arch = _arch(c)
        a = (torch.arange(c["res"], device=DEV, dtype=F64) / (c["res"] - 1)).float().double()
        z, y, x = torch.meshgrid(a, a, a, indexing="ij")
        pts = torch.stack([x.reshape(-1), y.reshape(-1), z.reshape(-1)], 1)
        p = _params(arch, _gen(seed, 1)).double()
        with torch.no_grad():
            return torch.cat([_net(arch, p, q)[0] for q in pts.split(CHUNK)]).reshape(z.shape)
    if kind == "batch":
        return _exact_batch(c, seed)
    if kind == "reptile":
        return _exact_reptile(c, seed)
    pose, rays, prior, params, g = _inputs(c, seed)
    spec = _spec(c)
    samp = _sample64(spec, rays, pose[0], prior)
    if kind == "sample":
        return dict(ray_obj=samp[0], t=samp[1], dt=samp[2], bins=None, flags=None)
    arch = _arch(c)
    if kind == "view":
        out, _ = _render64(arch, params, samp)
        return dict(rgb=out["rgb"], depth=out["depth"], opacity=out["opacity"])
    n = c["rays"]
    if kind == "autograd":
        out, grad = _render64(arch, params, samp, _mse_loss(rays, n, 0.1, 0.0), True)
        return dict(out, grad=grad * (_scale(c) or 1.0))  # the gradient carries the loss scale
    out, grad = _render64(arch, params, samp, _mse_loss(rays, n, c["lambda_d"], c["lambda_sigma"]), True)
    mom = _Moments(arch.n_params)
    _moments(mom, n, g)
    p, m = _adam64(params, grad, mom.adam_m, mom.adam_v)
    return dict(out, loss=out["loss"].reshape(1), params=p, adam_m=m)


def _exact_batch(c, seed):
    total = c["rays"] * BATCH_SPEC.n_samples
    if total > MOST_FWD:
        return None
    grad = total <= MOST_GRAD
    objs, rays, params, g = _batch_inputs(c, seed)
    outs, at, off, spans, grads = [], 0, 0, [], []
    for o, p in zip(objs, params):
        r = {k: v[at:at + o.n_rays] for k, v in rays.items()}
        samp = _sample64(BATCH_SPEC, r, o.world_to_obj, o.prior)
        out, gr = _render64(o.arch, p, samp, _mse_loss(r, o.n_rays, 0.0, 0.0), grad)
        outs.append(out)
        grads.append(gr)
        spans.append(off)
        at += o.n_rays
        off += -(-p.numel() // 64) * 64
    res = {k: torch.cat([x[k].reshape(-1) if k == "loss" else x[k] for x in outs]) for k in outs[0]}
    if not grad:
        return dict(res, params=None, adam_m=None)
    mom = _Moments(off)
    _moments(mom, c["rays"] / c["objects"], g)
    p64, g64 = torch.zeros(off, device=DEV, dtype=F64), torch.zeros(off, device=DEV, dtype=F64)
    for k, p, gr in zip(spans, params, grads):
        p64[k:k + p.numel()], g64[k:k + p.numel()] = p, gr
    p64, m64 = _adam64(p64, g64, mom.adam_m, mom.adam_v)
    return dict(res, params=p64, adam_m=m64)


def _exact_reptile(c, seed):
    g, rng = _gen(seed, 1), np.random.default_rng([seed, 2])
    arch, pose, n = _arch(c), _pose(rng), c["rays"]
    theta = _params(arch, g).double()
    rays = [_rays(n, c["fine"], pose, g) for _ in range(c["tasks"])]
    outs, step = [], torch.zeros_like(theta)
    for r in rays:
        samp, p = _sample64(_spec(c), r, pose[0], None), theta
        for _ in range(c["inner_steps"]):
            out, grad = _render64(arch, p, samp, _mse_loss(r, n, 0.0, 0.0), True)
            p = p - INNER_LR * grad
        outs.append(out)
        step += p - theta
    res = {k: torch.cat([x[k].reshape(-1) if k == "loss" else x[k] for x in outs]) for k in outs[0]}
    return dict(res, theta=theta + META_STEP * step / c["tasks"])


def _exact_yaw(c, seed):
    pts, prior = _cloud(c, seed)
    p = pts.double()
    scores, ext, cen = [], [], []
    for k in range(c["yaws"]):
        a = 2.0 * math.pi * k / c["yaws"]
        q = torch.stack([math.cos(a) * p[:, 0] - math.sin(a) * p[:, 1], math.sin(a) * p[:, 0] + math.cos(a) * p[:, 1],
                         p[:, 2]], 1)
        lo, hi = q.amin(0), q.amax(0)
        ext.append(hi - lo)
        cen.append(0.5 * (hi + lo))
        scores.append(_lookup(prior, (q - cen[-1]) / ext[-1] + 0.5).sum())
    return dict(scores=torch.stack(scores), extents=torch.stack(ext), centers=torch.stack(cen), best=None)
