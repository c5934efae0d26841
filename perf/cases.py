"""The work that is timed: calls a GaussianVideo program makes, over their range.

``listed()`` names the cases, ``draw(rng)`` gives one more of the same ranges,
``prepare`` makes what a program holds before the call, ``run`` is one pass
through the public entry points, ``work`` the bytes and operations a pass
cannot do without, and ``exact`` the pass's outputs in 64 bits by plain torch.

A case is a dict of plain values.  ``kind`` is the call:

* ``frame``       one frame forward and backward (render_fwd, render_bwd), the
                  step of a program that visits its frames one at a time;
* ``graph``       a whole clip, forward and backward, captured once (BatchGraph);
* ``clip``        the same as an eager call (render_batch), buffers kept;
* ``autograd``    the clip as a torch function with a torch loss
                  (RasterizeClip, RasterizeDynamicClip);
* ``render``      a clip rendered only (viewing a learned video);
* ``visibility``  per-Gaussian visibility counts over a clip;
* ``pyramid``     Gaussian pyramid of the target frames;
* ``adan``        one optimizer step over all parameters of a scene;
* ``ode``         camera ODE forward and its adjoint.

Scenes follow the repository's synthetic recipe: means uniform in a box in
front of the camera, normal log-scales, random rotations, normal opacity
logits, uniform colours; a smooth camera path; targets uniform in [0, 1].
"""
from __future__ import annotations

import math

import numpy as np
import torch

TILE = 16


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def _case(name, kind, **kw):
    c = dict(kind=kind, width=960, height=540, n=200_000, frames=50, dtype="f32", log_scale=-4.5,
             log_scale_std=0.5, z_near=2.0, z_far=10.0, moving=True, cubic=False, n_ctrl=0, poly_cov=False, sh=0)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # smallest step: a thumbnail frame with a few Gaussians; latency and launches
        _case("frame128_n2k", "frame", width=128, height=128, n=2000, frames=1, log_scale=-3.5, log_scale_std=0.3,
              z_far=6.0, moving=False),
        # an ordinary frame of a program that visits one frame per step
        _case("frame540p_n100k", "frame", n=100_000, frames=1, moving=False),
        # the fitting step: 50 shared-Gaussian frames with the fused L2 loss, one graph launch
        _case("clip540p_f50_n200k", "graph"),
        # the large clip: 1080p, bf16 parameters, cubic means, fixed camera
        _case("clip1080p_f32_n500k_bf16", "clip", width=1920, height=1080, n=500_000, frames=32, dtype="bf16",
              cubic=True, moving=False),
        # fitting with B-spline means and cubic scales and rotations (Eq. 2-3)
        _case("clip540p_f50_n200k_dyn", "clip", n_ctrl=8, poly_cov=True),
        # fitting with view-dependent colour
        _case("clip540p_f50_n200k_sh3", "graph", sh=3),
        # a torch training loop with its own loss on a short 480p clip of ragged size
        _case("autograd479p_f12_n61k", "autograd", width=853, height=479, n=61_003, frames=12),
        # viewing: frames of a learned video (400k Gaussians), no gradients
        _case("render540p_f24_n400k", "render", n=400_000, frames=24),
        # finding the Gaussians that no frame shows
        _case("visibility540p_f50_n200k", "visibility"),
        # spatial hierarchy: pyramid of a clip's targets
        _case("pyramid540p_f50_l4", "pyramid", levels=4),
        # optimizer step over a scene of 400k Gaussians
        _case("adan_n400k", "adan", n=400_000, frames=1),
        # learned camera: 100 poses by RK4 and their adjoint
        _case("ode_f100_s4", "ode", frames=100, substeps=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "frame", "graph", "graph", "clip", "clip", "autograd", "render", "visibility",
                       "pyramid", "adan", "ode"])
    if kind == "ode":
        return _case(None, kind, frames=_log_int(rng, 9, 200), substeps=rng.randint(1, 6))
    if kind == "adan":
        return _case(None, kind, n=_log_int(rng, 2000, 500_000), frames=1, cubic=rng.random() < 0.3,
                     sh=rng.choice([0, 0, 1, 3]))
    width = _log_int(rng, 96, 1920)
    height = max(64, int(width * rng.uniform(0.5, 1.0)))
    if kind == "pyramid":
        return _case(None, kind, width=width, height=height, n=0, levels=rng.randint(2, 6),
                     frames=max(1, min(64, int(rng.uniform(0.1, 1.0) * 26e6 / (width * height)))))
    # Gaussians in proportion to the frame, their size set by how many footprints cover a pixel
    n = max(500, min(500_000, int(width * height * rng.uniform(0.1, 0.45))))
    most = min(60.0, 16e6 / n, 50e6 / (width * height))
    frames = 1 if kind == "frame" else _log_int(rng, 2, max(3.0, most))
    z_far = rng.choice([6.0, 10.0])
    covered = rng.uniform(6.0, 80.0)
    size = max(0.35, covered * width * height / (n * 9.0 * math.pi) - 0.3)  # pixels squared
    log_scale = round(0.5 * math.log(size * 2.0 * z_far / width ** 2) - 0.125, 3)
    c = _case(None, kind, width=width, height=height, n=n, frames=frames, dtype=rng.choice(["f32", "f32", "bf16"]),
              z_far=z_far, log_scale=log_scale, moving=rng.random() < 0.7)
    if kind != "frame":
        form = rng.choice(["static", "static", "cubic", "dynamic", "sh"])
        c["cubic"] = form == "cubic"
        if form == "dynamic":
            c["n_ctrl"], c["poly_cov"] = rng.choice([4, 6, 8, 12]), True
        if form == "sh":
            c["sh"] = rng.choice([1, 2, 3])
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

N_THETA = 5191


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)


def _uniform(g, shape, lo=0.0, hi=1.0):
    return torch.rand(shape, generator=g, device="cuda") * (hi - lo) + lo


def _normal(g, shape, mean=0.0, std=1.0):
    return torch.randn(shape, generator=g, device="cuda") * std + mean


def _scene_tensors(c, g):
    n = c["n"]
    p = dict(means=torch.stack([_uniform(g, n, -1, 1), _uniform(g, n, -1, 1), _uniform(g, n, c["z_near"], c["z_far"])]),
             log_scales=_normal(g, (3, n), c["log_scale"], c["log_scale_std"]),
             quats=torch.nn.functional.normalize(_normal(g, (4, n)), dim=0),
             opacity_logits=_normal(g, n), colors=_uniform(g, (3, n)))
    if c["cubic"]:
        p["mean_coeffs"] = _normal(g, (3, 3, n), 0, 0.05)
    if c["n_ctrl"]:
        p["ctrl"] = p["means"][None] + _normal(g, (c["n_ctrl"], 3, n), 0, 0.05)
    if c["poly_cov"]:
        p["scale_coeffs"] = _normal(g, (3, 3, n), 0, 0.05)
        p["quat_coeffs"] = _normal(g, (3, 4, n), 0, 0.05)
    if c["sh"]:
        p["sh"] = _normal(g, ((c["sh"] + 1) ** 2 - 1, 3, n), 0, 0.1)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    return {k: v.to(dt).contiguous() for k, v in p.items()}


def _poses(c, seed):
    """World->camera poses: the identity, or sums of three sinusoids per axis and a slow rotation of up to 10 degrees."""
    F = c["frames"]
    out = np.zeros((F, 7))
    out[:, 0] = 1.0
    if c["moving"]:
        rng = np.random.default_rng(int(seed) + 5)
        f = np.arange(F)
        period, phase = rng.uniform(20.0, 80.0, (3, 3)), rng.uniform(0.0, 2 * math.pi, (3, 3))
        for axis in range(3):
            out[:, 4 + axis] = sum(0.2 * np.sin(2 * math.pi * f / period[axis, k] + phase[axis, k]) for k in range(3))
        axis = rng.normal(size=3)
        half = np.radians(rng.uniform(1.0, 10.0)) * (f / max(1, F - 1) - 0.5) / 2
        out[:, 0], out[:, 1:4] = np.cos(half), np.sin(half)[:, None] * axis / np.linalg.norm(axis)
    return torch.from_numpy(out.astype(np.float32)).cuda()


def _times(c):
    F = c["frames"]
    return torch.from_numpy((np.arange(F) / max(1, F - 1)).astype(np.float32)).cuda()


def _targets(c, g):
    return _uniform(g, (c["frames"], 3, c["height"], c["width"]))


def _ode_inputs(c, g):
    parts = []
    for fan_out, fan_in, scale in ((64, 8, 1.0), (64, 64, 1.0), (7, 64, 0.1)):
        b = scale / math.sqrt(fan_in)
        parts += [_uniform(g, fan_out * fan_in, -b, b), _uniform(g, fan_out, -b, b)]
    z0 = torch.cat([torch.tensor([1.0, 0.0, 0.0, 0.0], device="cuda"), torch.zeros(3, device="cuda")])
    z0 = z0 + _normal(g, 7, 0, 0.1)
    return torch.cat(parts), z0, _normal(g, (c["frames"], 7))


def _adan_inputs(c, g):
    params = {k: v.float() for k, v in _scene_tensors(c, g).items()}
    grads = [{k: _normal(g, v.shape, 0, 1e-3) for k, v in params.items()} for _ in range(3)]
    return params, grads


# ---------------------------------------------------------------------------
# what a program holds, and one pass
# ---------------------------------------------------------------------------

def prepare(case, seed):
    from paper_2501_04782_amd import camera, optim, raster
    c, g = case, _generator(seed)
    if c["kind"] == "ode":
        theta, z0, up = _ode_inputs(c, g)
        ws = camera.OdeWorkspace(c["frames"], c["substeps"])
        return dict(kind="ode", theta=theta.requires_grad_(), z0=z0.requires_grad_(), up=up, ws=ws, c=c)
    if c["kind"] == "pyramid":
        return dict(kind="pyramid", images=_targets(c, g), levels=c["levels"])
    if c["kind"] == "adan":
        params, grads = _adan_inputs(c, g)
        opt = optim.Adan(list(params.values()))
        for k in range(2):  # past the first steps, which have no history
            opt.step(list(grads[k].values()))
        return dict(kind="adan", opt=opt, grads=list(grads[2].values()))
    params = _scene_tensors(c, g)
    poses, times, targets = _poses(c, seed), _times(c), _targets(c, g)
    cam = raster.Camera(c["width"], c["height"], float(c["width"]), float(c["width"]), c["width"] / 2, c["height"] / 2)
    scene = raster.Scene(**params)
    F = c["frames"]
    ws = raster.Workspace(cam, scene.n, F, raster.estimate_capacity(scene, cam, poses, times, margin=1.25))
    s = dict(kind=c["kind"], scene=scene, cam=cam, poses=poses, times=times, targets=targets, ws=ws, c=c)
    if c["kind"] == "graph":
        s["graph"] = raster.BatchGraph(scene, cam, poses, times, ws, targets=targets)
    elif c["kind"] == "autograd":
        s["leaves"] = {k: v.requires_grad_() for k, v in params.items()}
        s["poses"].requires_grad_()
    else:
        s["images"] = torch.empty(F, 3, c["height"], c["width"], device="cuda")
    if c["kind"] in ("frame", "clip"):
        s["grads"] = raster.grad_buffers(scene)
        s["dposes"] = torch.empty(F, 7, device="cuda")
    if c["kind"] == "frame":
        s["T"] = torch.empty(c["height"], c["width"], device="cuda")
    if c["kind"] == "clip":
        s["loss"] = torch.empty(F, device="cuda")
    return s


def run(state):
    from paper_2501_04782_amd import camera, raster
    s = state
    kind = s["kind"]
    if kind == "frame":
        scene, cam, pose = s["scene"], s["cam"], s["poses"][0]
        raster.render_fwd(scene, cam, pose, 0.0, s["ws"], image=s["images"][0], T_final=s["T"])
        raster.render_bwd(scene, cam, pose, 0.0, s["ws"], s["images"][0], target=s["targets"][0],
                          loss_scale=2.0 / (3.0 * cam.width * cam.height), grads=s["grads"],
                          dL_dpose7=s["dposes"][0])
        return dict(images=s["images"], T=s["T"], grads=s["grads"], dposes=s["dposes"])
    if kind == "graph":
        s["graph"].launch()
        b = s["graph"]
        return dict(images=b.images, loss=b.loss, grads=b.grads, dposes=b.dL_dposes)
    if kind == "clip":
        r = raster.render_batch(s["scene"], s["cam"], s["poses"], s["times"], s["ws"], targets=s["targets"],
                                images=s["images"], loss=s["loss"], grads=s["grads"], dL_dposes=s["dposes"])
        return dict(images=r["images"], loss=r["loss"], grads=r["grads"], dposes=r["dL_dposes"])
    if kind == "autograd":
        p = s["leaves"]
        for v in list(p.values()) + [s["poses"]]:
            v.grad = None
        if "ctrl" in p:
            images = raster.RasterizeDynamicClip.apply(
                p["ctrl"], p["log_scales"], p["quats"], p["opacity_logits"], p["colors"], p.get("scale_coeffs"),
                p.get("quat_coeffs"), s["poses"], s["times"], s["cam"], s["ws"])
        else:
            images = raster.RasterizeClip.apply(
                p["means"], p["log_scales"], p["quats"], p["opacity_logits"], p["colors"], p.get("mean_coeffs"),
                p.get("sh"), s["poses"], s["times"], s["cam"], s["ws"])
        loss = ((images - s["targets"]) ** 2).mean()
        loss.backward()
        return dict(images=images.detach(), loss=loss.detach(), grads={k: v.grad for k, v in p.items()},
                    dposes=s["poses"].grad)
    if kind == "render":
        r = raster.render_batch(s["scene"], s["cam"], s["poses"], s["times"], s["ws"], backward=False,
                                images=s["images"])
        return dict(images=r["images"])
    if kind == "visibility":
        counts = raster.visibility_counts(s["scene"], s["cam"], s["poses"], s["times"], s["ws"], images=s["images"])
        return dict(counts=counts, images=s["images"])
    if kind == "pyramid":
        return dict(levels=raster.gaussian_pyramid(s["images"], s["levels"])[1:])
    if kind == "adan":
        s["opt"].step(s["grads"])
        return dict(params=s["opt"].params, states=s["opt"].states)
    if kind == "ode":
        c = s["c"]
        s["theta"].grad = s["z0"].grad = None
        poses = camera.CameraODE.apply(s["theta"], s["z0"], c["frames"], c["substeps"], s["ws"])
        poses.backward(s["up"])
        return dict(poses=poses.detach(), dtheta=s["theta"].grad, dz0=s["z0"].grad)
    raise ValueError(kind)


def work(case):
    c = case
    F, n, P = c["frames"], c["n"], c["width"] * c["height"]
    if c["kind"] == "ode":
        evals = (F - 1) * c["substeps"] * 4
        macs = 8 * 64 + 64 * 64 + 64 * 7
        return dict(bytes=4.0 * (2 * N_THETA + 14 * F), flops=evals * macs * 6.0)
    per = 14 + (9 if c["cubic"] else 0) + (3 * c["n_ctrl"] - 3 if c["n_ctrl"] else 0) + (21 if c["poly_cov"] else 0)
    per += 3 * ((c["sh"] + 1) ** 2 - 1)
    if c["kind"] == "adan":
        return dict(bytes=44.0 * per * n, flops=20.0 * per * n)
    if c["kind"] == "pyramid":
        total, h, w = F * 3 * P, c["height"], c["width"]
        read = F * 3 * P
        for level in range(1, c["levels"]):
            h, w = (h + 1) // 2, (w + 1) // 2
            total += F * 3 * h * w
        return dict(bytes=4.0 * total, flops=30.0 * (total - read))
    # contributors per pixel: footprints of the 3-sigma ellipses over a pixel, fewer once they saturate it
    size = c["width"] ** 2 * math.exp(2 * c["log_scale"] + c["log_scale_std"] ** 2) / (c["z_near"] * c["z_far"])
    covered = 9.0 * math.pi * (size + 0.3) * n / P
    pairs = covered / (1.0 + covered / 80.0) * P * F
    read = per * n * (2 if c["dtype"] == "bf16" else 4)
    if c["kind"] == "render":
        return dict(bytes=read + 12.0 * P * F, flops=25.0 * pairs)
    if c["kind"] == "visibility":
        return dict(bytes=read + 12.0 * P * F + 4.0 * n, flops=25.0 * pairs)
    return dict(bytes=read + 4.0 * per * n + 24.0 * P * F, flops=95.0 * pairs)


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _spline_basis(M, t):
    """Clamped cubic B-spline basis N_0..N_{M-1} at t (Cox-de Boor)."""
    u = [0.0] * 4 + [k / (M - 3) for k in range(1, M - 3)] + [1.0] * 4
    span = M - 1 if t >= 1.0 else max(j for j in range(3, M) if u[j] <= t)
    N = [1.0 if j == span else 0.0 for j in range(M + 3)]
    for p in range(1, 4):
        N = [((t - u[j]) / (u[j + p] - u[j]) * N[j] if u[j + p] > u[j] else 0.0) +
             ((u[j + p + 1] - t) / (u[j + p + 1] - u[j + 1]) * N[j + 1] if u[j + p + 1] > u[j + 1] else 0.0)
             for j in range(M + 3 - p)]
    return N[:M]


def _sh_basis(degree, x, y, z):
    """Real orthonormal spherical harmonics of degrees 1..degree."""
    pi = math.pi
    a = math.sqrt(3 / (4 * pi))
    Y = [-a * y, a * z, -a * x]
    if degree >= 2:
        b, e = math.sqrt(15 / (4 * pi)), math.sqrt(5 / (16 * pi))
        Y += [b * x * y, -b * y * z, e * (2 * z * z - x * x - y * y), -b * x * z, b / 2 * (x * x - y * y)]
    if degree >= 3:
        h, k = math.sqrt(35 / (32 * pi)), math.sqrt(105 / (4 * pi))
        m, o = math.sqrt(21 / (32 * pi)), math.sqrt(7 / (16 * pi))
        r = 4 * z * z - x * x - y * y
        Y += [-h * y * (3 * x * x - y * y), k * x * y * z, -m * y * r, o * z * (2 * z * z - 3 * x * x - 3 * y * y),
              -m * x * r, k / 2 * z * (x * x - y * y), -h * x * (x * x - 3 * y * y)]
    return Y


def _rotation(q):
    w, x, y, z = q
    one = torch.ones_like(w)
    return [[one - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
            [2 * (x * y + w * z), one - 2 * (x * x + z * z), 2 * (y * z - w * x)],
            [2 * (x * z - w * y), 2 * (y * z + w * x), one - 2 * (x * x + y * y)]]


def _project(c, p, intr, pose, t):
    """Centre, conic, opacity and colour of every Gaussian in one frame ([9, n]), its depth, its footprint's half-extents
    and whether it is in front of the camera."""
    if "ctrl" in p:
        mu = sum(w * p["ctrl"][i] for i, w in enumerate(_spline_basis(c["n_ctrl"], t)) if w != 0.0)
    else:
        mu = p["means"]
    if "mean_coeffs" in p:
        mu = mu + sum(p["mean_coeffs"][k] * t ** (k + 1) for k in range(3))
    ls, q = p["log_scales"], p["quats"]
    if "scale_coeffs" in p:
        ls = ls + sum(p["scale_coeffs"][k] * t ** (k + 1) for k in range(3))
        q = q + sum(p["quat_coeffs"][k] * t ** (k + 1) for k in range(3))
    R = _rotation(q / q.norm(dim=0, keepdim=True))
    s = ls.exp()
    Rc = _rotation(pose[:4] / pose[:4].norm())
    tc = pose[4:]
    m = [((tc[i] + Rc[i][0] * mu[0]) + Rc[i][1] * mu[1]) + Rc[i][2] * mu[2] for i in range(3)]
    front = m[2] > 0.01
    m[2] = torch.where(front, m[2], torch.ones_like(m[2]))
    fx, fy, cx, cy = intr
    u, v = fx * m[0] / m[2] + cx, fy * m[1] / m[2] + cy
    J = [[fx / m[2], None, -fx * m[0] / m[2] ** 2], [None, fy / m[2], -fy * m[1] / m[2] ** 2]]
    W = [[J[0][0] * Rc[0][j] + J[0][2] * Rc[2][j] for j in range(3)],
         [J[1][1] * Rc[1][j] + J[1][2] * Rc[2][j] for j in range(3)]]
    V = [[sum(W[i][k] * R[k][j] for k in range(3)) * s[j] for j in range(3)] for i in range(2)]
    c00 = sum(V[0][j] ** 2 for j in range(3)) + 0.3
    c01 = sum(V[0][j] * V[1][j] for j in range(3))
    c11 = sum(V[1][j] ** 2 for j in range(3)) + 0.3
    det = c00 * c11 - c01 * c01
    col = [p["colors"][k] for k in range(3)]
    if "sh" in p:
        d = torch.stack([mu[i] + sum(Rc[j][i] * tc[j] for j in range(3)) for i in range(3)])
        d = d / d.norm(dim=0, keepdim=True)
        Y = _sh_basis(c["sh"], d[0], d[1], d[2])
        col = [col[k] + sum(y * p["sh"][i][k] for i, y in enumerate(Y)) for k in range(3)]
    proj = torch.stack([u, v, c11 / det, -c01 / det, c00 / det, torch.sigmoid(p["opacity_logits"])] + col)
    with torch.no_grad():
        box = torch.stack([3 * c00.sqrt(), 3 * c11.sqrt()]) * 1.0001 + 0.01
    return proj, m[2].detach(), box, front


def _candidates(c, proj, depth, box, front):
    """(tile, Gaussian) pairs whose footprint box meets the tile, by tile and then by (fp32 depth, index)."""
    tx, ty = -(-c["width"] // TILE), -(-c["height"] // TILE)
    lo = ((proj[:2] - box - (TILE - 0.5)) / TILE).ceil().clamp(min=0)
    hi = ((proj[:2] + box - 0.5) / TILE).floor()
    hi = torch.minimum(hi, torch.tensor([[tx - 1.0], [ty - 1.0]], device=hi.device, dtype=hi.dtype))
    span = (hi - lo + 1).clamp(min=0) * front
    span = span.long()
    count = span[0] * span[1]
    order = torch.sort(depth.float(), stable=True).indices
    rank = torch.empty_like(order)
    rank[order] = torch.arange(len(order), device=order.device)
    gid = torch.repeat_interleave(torch.arange(len(order), device=order.device), count)
    first = torch.repeat_interleave(torch.cumsum(count, 0) - count, count)
    cell = torch.arange(len(gid), device=gid.device) - first
    w = span[0][gid]
    tile = (lo[1][gid].long() + cell // w) * tx + lo[0][gid].long() + cell % w
    tile, by = torch.sort(tile * len(order) + rank[gid])
    return torch.div(tile, len(order), rounding_mode="floor"), gid[by], tx * ty, tx


def _composite(c, proj, tiles, gids, tx, target, scale, image, T):
    """Composite the given tiles (gids [tiles, entries], -1 past a tile's end) into image and T; the gradient of
    scale / 2 * sum (image - target)^2 is added to proj.grad."""
    W, H = c["width"], c["height"]
    pad = torch.cat([proj, torch.zeros(9, 1, dtype=proj.dtype, device=proj.device)], 1)  # entry -1: opacity 0
    e = pad[:, gids.reshape(-1)].reshape(9, *gids.shape, 1)
    px = torch.arange(TILE * TILE, device=proj.device)
    x = (tiles % tx * TILE)[:, None] + px % TILE
    y = torch.div(tiles, tx, rounding_mode="floor")[:, None] * TILE + torch.div(px, TILE, rounding_mode="floor")
    inside = (x < W) & (y < H)
    dx, dy = (x + 0.5)[:, None] - e[0], (y + 0.5)[:, None] - e[1]
    q = e[2] * dx * dx + 2 * e[3] * dx * dy + e[4] * dy * dy
    alpha = (e[5] * torch.exp(-0.5 * q)).clamp(max=0.99)
    alpha = torch.where((q <= 9.0) & (alpha >= 1.0 / 255.0), alpha, torch.zeros_like(alpha))
    after = torch.exp(torch.cumsum(torch.log1p(-alpha), 1))
    alive = after >= 1e-4
    w = torch.where(alive, alpha * torch.cat([torch.ones_like(after[:, :1]), after[:, :-1]], 1),
                    torch.zeros_like(alpha))
    colour = torch.stack([(w * e[6 + k]).sum(1) for k in range(3)])
    x, y = x[inside], y[inside]
    got = colour[:, inside]
    with torch.no_grad():
        image[:, y, x] = got
        T[y, x] = torch.where(alive, 1 - alpha, torch.ones_like(alpha)).prod(1)[inside]
    if proj.requires_grad:
        (0.5 * scale * ((got - target[:, y, x].double()) ** 2).sum()).backward()


def _render(c, proj, depth, box, front, target, scale):
    """Image and final transmittance of one frame; gradients go to proj.grad."""
    H, W = c["height"], c["width"]
    image = torch.zeros(3, H, W, dtype=torch.float64, device="cuda")
    T = torch.ones(H, W, dtype=torch.float64, device="cuda")
    with torch.no_grad():
        tile, gid, n_tiles, tx = _candidates(c, proj, depth, box, front)
        count = torch.bincount(tile, minlength=n_tiles)
        start = torch.cumsum(count, 0) - count
        length, order = torch.sort(count, descending=True)
    lengths = length.tolist()
    at = 0
    while at < n_tiles and lengths[at] > 0:
        many = max(1, int(6e6 // (lengths[at] * TILE * TILE)))
        tiles = order[at:at + many]
        k = torch.arange(lengths[at], device="cuda")
        where = (start[tiles][:, None] + k).clamp(max=len(gid) - 1)
        gids = torch.where(k < count[tiles][:, None], gid[where], torch.full_like(where, proj.shape[1]))
        _composite(c, proj, tiles, gids, tx, target, scale, image, T)
        at += many
    return image, T


def _exact_clip(c, seed):
    g = _generator(seed)
    backward = c["kind"] not in ("render", "visibility")
    p = {k: v.double().requires_grad_(backward) for k, v in _scene_tensors(c, g).items()}
    poses = _poses(c, seed).double().requires_grad_(backward)
    times = [0.0] * c["frames"] if c["kind"] == "frame" else _times(c).double().tolist()
    targets = _targets(c, g)
    F, H, W = c["frames"], c["height"], c["width"]
    intr = torch.tensor([W, W, W / 2, H / 2], dtype=torch.float64, device="cuda", requires_grad=backward)
    scale = 2.0 / (3.0 * H * W * F)
    images = torch.empty(F, 3, H, W, device="cuda", dtype=torch.float64)
    for f in range(F):
        with torch.set_grad_enabled(backward):
            proj, depth, box, front = _project(c, p, intr, poses[f], times[f])
            leaf = proj.detach().requires_grad_(backward)
            images[f], T = _render(c, leaf, depth, box, front, targets[f], scale)
            if backward:
                leaf.grad[:, ~front] = 0
                proj.backward(leaf.grad)
    if not backward:
        return dict(images=images) if c["kind"] == "render" else dict(counts=None, images=images)
    loss = torch.stack([0.5 * scale * ((images[f] - targets[f].double()) ** 2).sum() for f in range(F)])
    grads = {k: v.grad for k, v in p.items()}
    if c["kind"] == "autograd":
        if "ctrl" in p:
            grads["means"] = None
        return dict(images=images, loss=loss.sum(), grads=grads, dposes=poses.grad)
    grads["intrinsics"] = intr.grad
    if "ctrl" in p:
        grads["means"] = None
    if c["kind"] == "frame":
        return dict(images=images, T=T, grads=grads, dposes=poses.grad)
    return dict(images=images, loss=loss, grads=grads, dposes=poses.grad)


def _exact_pyramid(c, seed):
    x = _targets(c, _generator(seed)).double()
    x = x.reshape(-1, 1, *x.shape[-2:])
    k = torch.tensor([1.0, 4.0, 6.0, 4.0, 1.0], dtype=torch.float64, device="cuda") / 16
    out, F = [], c["frames"]
    for _ in range(1, c["levels"]):
        x = torch.nn.functional.pad(x, (2, 2, 2, 2), mode="reflect")
        h, w = x.shape[-2:]
        rows = sum(k[i] * x[:, :, i:h - 4 + i:2] for i in range(5))
        x = sum(k[i] * rows[:, :, :, i:w - 4 + i:2] for i in range(5))
        out.append(x.reshape(F, 3, *x.shape[-2:]))
    return dict(levels=out)


def _exact_adan(c, seed):
    params, grads = _adan_inputs(c, _generator(seed))
    b1, b2, b3 = 0.02, 0.08, 0.01
    out, states = [], []
    for key, p in params.items():
        p, prev = p.double(), None
        for k in range(3):
            g = grads[k][key].double()
            d = torch.zeros_like(g) if prev is None else g - prev
            if k == 0:
                m, v, n = g, torch.zeros_like(g), g * g
            else:
                m = (1 - b1) * m + b1 * g
                v = d if k == 1 else (1 - b2) * v + b2 * d
                n = (1 - b3) * n + b3 * (g + (1 - b2) * d) ** 2
            p = p - 0.01 * 0.99995 ** k / (n + 1e-8).sqrt() * (m + (1 - b2) * v)
            prev = g
        out.append(p)
        states.append(torch.stack([m, v, n, prev]))
    return dict(params=out, states=states)


def _exact_ode(c, seed):
    theta, z0, up = (v.double().cpu() for v in _ode_inputs(c, _generator(seed)))
    theta.requires_grad_()
    z0.requires_grad_()
    W1, b1, W2, b2, W3, b3 = torch.split(theta, [512, 64, 4096, 64, 448, 7])
    W1, W2, W3 = W1.view(64, 8), W2.view(64, 64), W3.view(7, 64)

    def field(z, t):
        h = torch.tanh(W1 @ torch.cat([z, torch.tensor([t], dtype=torch.float64)]) + b1)
        return W3 @ torch.tanh(W2 @ h + b2) + b3

    F, S = c["frames"], c["substeps"]
    h, z = 1.0 / (S * (F - 1)), z0
    poses = [z]
    for f in range(1, F):
        for s in range(S):
            t = ((f - 1) * S + s) * h
            k1 = field(z, t)
            k2 = field(z + 0.5 * h * k1, t + 0.5 * h)
            k3 = field(z + 0.5 * h * k2, t + 0.5 * h)
            k4 = field(z + h * k3, t + h)
            z = z + h / 6 * (k1 + 2 * k2 + 2 * k3 + k4)
        poses.append(z)
    poses = torch.stack([torch.cat([z[:4] / z[:4].norm(), z[4:]]) for z in poses])
    poses.backward(up)
    return dict(poses=poses.detach(), dtheta=theta.grad, dz0=z0.grad)


def exact(case, seed):
    c = case
    if c["kind"] == "ode":
        return _exact_ode(c, seed)
    if c["kind"] == "pyramid":
        return _exact_pyramid(c, seed)
    if c["kind"] == "adan":
        return _exact_adan(c, seed)
    return _exact_clip(c, seed)
