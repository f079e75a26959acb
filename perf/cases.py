"""The workloads that this package is timed on, from the smallest call to the largest.

Every case goes through the public entry points as a SLAM program calls them:

  track     one tracking iteration (Eq. 2 of the paper): render, masked loss, pose gradient, pose step
  loop      one tracking/mapping iteration with the plain L1 and the fused backward and Adam step
  map       one submap-update iteration: L1 + SSIM + depth loss, isotropic regulariser, full backward, Adam
  render    a submap rendered at several keyframes (forward only)
  grad      the differentiable render under PyTorch autograd, with a loss of the caller's own
  register  one loop edge: every keyframe of two submaps localised in the other, and the fusion
  overlap   the overlap ratio of two submaps (loop detection)
  prune     opacity pruning of a submap and of its optimiser state
  adjust    the map adjustment after pose-graph optimisation

Sizes are those of the package's own benchmark and tests (4,096 Gaussians at 160x120, 200k at 1200x680, the
150k + 120k pair, 64 submaps of 200k) and ragged ones between them.  Optimiser state is that of a run under way:
moments left by earlier, larger gradients and learning rates decayed a hundredfold, so that a state can be stepped
many times without the scene moving away.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2408_10154_amd import synth
from paper_2408_10154_amd.register import default_params, register_pair
from paper_2408_10154_amd.render import (GaussianSet, RenderBatch, adam, adjust_submaps, loss_isotropic,
                                         overlap_ratio, prune_gaussians, render)

DEV = "cuda"
FIELDS = GaussianSet.FIELDS
LR = dict(mean=1e-5, log_scale=5e-5, quat=1e-5, opacity_logit=5e-4, rgb=2.5e-5)  # decayed mapping rates
LR_ROT, LR_TRANS = 2e-5, 1e-4                                                    # decayed tracking rates
STEP0 = 100                                                                      # Adam steps taken before
BG = (0.1, 0.2, 0.3)


def listed():
    return [
        # the smallest iteration that a program runs: latency and launches count
        dict(name="track_4096_160x120", kind="track", box="cube", n=4096, width=160, height=120, focal=150.0),
        # frame-to-model tracking at a 640x480 sensor, ragged submap size
        dict(name="track_97k_640x480", kind="track", box="room", n=97_003, width=640, height=480, focal=500.0),
        # the package's benchmark loop
        dict(name="loop_200k_1200x680", kind="loop", box="room", n=200_000, width=1200, height=680, focal=600.0),
        # the same submap under the whole mapping loss
        dict(name="map_200k_1200x680", kind="map", box="room", n=200_000, width=1200, height=680, focal=600.0),
        # mapping of a young submap on a cropped image
        dict(name="map_23k_317x211", kind="map", box="room", n=23_017, width=317, height=211, focal=180.0),
        # a submap rendered at its keyframes (views, targets, residuals)
        dict(name="render_150k_8x640x480", kind="render", n=150_000, views=8, width=640, height=480, focal=500.0),
        # a caller's own loss through autograd, odd image sides, with a background
        dict(name="grad_31k_333x251", kind="grad", box="room", n=31_001, width=333, height=251, focal=200.0),
        # loop edges: the benchmark pair with all its views, and two small submaps with two views each
        dict(name="register_150k_120k_8x8", kind="register", n_p=150_000, n_q=120_000, views=8, width=640,
             height=480, focal=500.0, iters=10),
        dict(name="register_21k_17k_2x2", kind="register", n_p=21_000, n_q=17_003, views=2, width=320, height=240,
             focal=250.0, iters=10),
        # loop detection between the benchmark pair's submaps, at an odometry estimate
        dict(name="overlap_150k_120k", kind="overlap", n_p=150_000, n_q=120_000, rot_deg=3.0, trans=0.1),
        # pruning of a submap with both Adam moments
        dict(name="prune_200k", kind="prune", n=200_000, threshold=0.5),
        # all submaps of a long sequence moved after pose-graph optimisation
        dict(name="adjust_64x200k", kind="adjust", n=200_000, submaps=64, poses=100),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["track", "loop", "map", "render", "grad", "register", "overlap", "prune", "adjust"])
    if kind in ("track", "loop", "map", "grad"):
        width = log_int(96, 1200)
        height = max(64, int(width * rng.uniform(0.55, 0.78)))
        small = rng.random() < 0.3
        return dict(kind=kind, box="cube" if small else "room", n=log_int(3000, 20_000 if small else 200_000),
                    width=width, height=height, focal=round(width * rng.uniform(0.5, 0.9), 1))
    if kind == "render":
        width = log_int(160, 800)
        return dict(kind=kind, n=log_int(5000, 150_000), views=rng.randint(1, 8), width=width,
                    height=int(width * rng.uniform(0.6, 0.76)), focal=round(width * rng.uniform(0.6, 0.85), 1))
    if kind == "register":
        width = log_int(160, 640)
        return dict(kind=kind, n_p=log_int(5000, 150_000), n_q=log_int(5000, 120_000), views=rng.randint(1, 8),
                    width=width, height=int(width * rng.uniform(0.6, 0.75)), focal=round(width * 0.78, 1),
                    iters=rng.randint(5, 10))
    if kind == "overlap":
        return dict(kind=kind, n_p=log_int(1500, 150_000), n_q=log_int(1500, 120_000),
                    rot_deg=round(rng.uniform(0.0, 4.0), 2), trans=round(rng.uniform(0.0, 0.15), 3))
    if kind == "prune":
        return dict(kind=kind, n=log_int(2000, 330_000), threshold=rng.choice([0.1, 0.3, 0.5]))
    return dict(kind="adjust", n=log_int(2000, 200_000), submaps=rng.randint(1, 64), poses=rng.randint(0, 150))


# ------------------------------------------------------------------ inputs

def _cam(case):
    return synth.camera(case["focal"], case["focal"], case["width"] / 2, case["height"] / 2, case["width"],
                        case["height"])


def _gauss(g):
    return {k: torch.as_tensor(np.ascontiguousarray(g[k], np.float32), device=DEV) for k in FIELDS}


def _volume(case, seed):
    """Gaussians filling a box before an identity camera, and a measurement from 2 degrees / 3 cm away with holes
    in its depth, as an RGB-D sensor has them."""
    rng = np.random.default_rng(seed)
    lo, hi = ((-1.0, -1.0, 1.5), (1.0, 1.0, 3.5)) if case["box"] == "cube" else ((-3.0, -1.5, 0.5), (3.0, 1.5, 4.5))
    g = _gauss(synth.gaussians_in_box(rng, case["n"], lo, hi))
    cam, w2c = _cam(case), synth.identity_w2c()
    pose = torch.as_tensor(synth.perturbation(rng, 2.0, 0.03), device=DEV)
    with torch.no_grad():
        rgb, depth, _ = _render_plain(g, cam, w2c, pose, torch.float32)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    depth = torch.where(torch.rand(depth.shape, generator=gen, device=DEV) < 0.05, torch.zeros_like(depth), depth)
    return g, cam, w2c, rgb, depth


def _submap(case, seed):
    """A room's surfaces as a submap, and keyframes inside the room."""
    rng = np.random.default_rng(seed)
    g = synth.gaussians_in_box(rng, case["n"], (0, 0, 0), (1, 1, 1))
    g["mean"] = synth.room_points(rng, case["n"]).astype(np.float32)
    half = np.array([3.0, 1.5, 2.0])
    views = []
    for _ in range(case["views"]):
        pos = rng.uniform(-0.35, 0.35, 3) * half
        target = rng.uniform(-1.0, 1.0, 3) * half
        target[rng.integers(2) * 2] *= 2.0
        c2w = synth.look_at_c2w(pos, target)
        w2c = np.concatenate([c2w[:3, :3].T, -c2w[:3, :3].T @ c2w[:3, 3:4]], 1).astype(np.float32)
        views.append(w2c)
    return _gauss(g), _cam(case), views


def _pair(case, seed):
    d = synth.registration_pair(seed, case["n_p"], case["n_q"], views_p=case.get("views", 1),
                                views_q=case.get("views", 1), width=case.get("width", 640),
                                height=case.get("height", 480), f=case.get("focal", 500.0), rot_deg_max=2.0,
                                trans_max=0.05, layout="x_split")
    return d, _gauss(d["P"]), _gauss(d["Q"])


def _moments(g, case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed + 7)
    s = 30.0 / (case["width"] * case["height"])
    out = {}
    for k in FIELDS:
        m = s * torch.randn(g[k].shape, generator=gen, device=DEV)
        v = (s * (0.5 + torch.rand(g[k].shape, generator=gen, device=DEV))) ** 2
        out[k] = (m, v, LR[k])
    return out


def _pose_state(seed):
    gen = torch.Generator(device=DEV).manual_seed(seed + 8)
    pose = torch.as_tensor(synth.identity_pose()[None], device=DEV).contiguous()
    m = 0.1 * torch.randn(1, 7, generator=gen, device=DEV)
    v = (0.1 * (0.5 + torch.rand(1, 7, generator=gen, device=DEV))) ** 2
    return pose, torch.zeros_like(pose), m, v


def _batch(gs, cam, views, pose):
    """A batch with half as much room again as its lists need now, so that no iteration waits for the host."""
    jobs = [(gs, cam, w) for w in views]
    b = RenderBatch(jobs)
    b.project(pose)
    b.bin_sort()
    room = int(b.instances() * 1.5) + 4096
    b.close()
    return RenderBatch(jobs, capacity=room, auto_grow=False)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("track", "loop", "map", "grad"):
        g, cam, w2c, rgb, depth = _volume(case, seed)
        gs = GaussianSet(**g)
        pose, pose_grad, pm, pv = _pose_state(seed)
        s = dict(kind=kind, gs=gs, batch=_batch(gs, cam, [w2c], pose), pose=pose, pose_grad=pose_grad, pm=pm, pv=pv,
                 rgb=rgb.reshape(-1), depth=depth.reshape(-1), step=STEP0)
        if kind == "grad":
            gen = torch.Generator(device=DEV).manual_seed(seed + 9)
            npix = case["width"] * case["height"]
            s["up"] = [torch.randn(k * npix, generator=gen, device=DEV) / npix for k in (3, 1, 1)]
            s["leaves"] = [pose] + gs.tensors()
            for t in s["leaves"]:
                t.requires_grad_(True)
        else:
            s["loss"] = torch.zeros(1, device=DEV)
            s["median"] = torch.zeros(1, device=DEV)
            s["g_rgb"], s["g_depth"] = torch.zeros_like(s["rgb"]), torch.zeros_like(s["depth"])
            s["scale"] = torch.zeros(1, device=DEV)
            s["pose_groups"] = [(pose[0, :4], pose_grad[0, :4], pm[0, :4], pv[0, :4], LR_ROT),
                                (pose[0, 4:], pose_grad[0, 4:], pm[0, 4:], pv[0, 4:], LR_TRANS)]
        if kind in ("loop", "map"):
            s["moments"] = _moments(g, case, seed)
        if kind == "loop":  # 1 / |Omega| of the measurement, once for all iterations on it
            s["batch"].loss_l1(s["rgb"], s["depth"], s["loss"], s["g_rgb"], s["g_depth"], s["scale"])
        if kind == "map":
            s["grads"] = gs.zeros_like()
            s["iso"] = torch.zeros(1, device=DEV)
            s["iso_work"] = torch.empty(256, device=DEV)
            s["groups"] = [(getattr(gs, k), getattr(s["grads"], k)) + s["moments"][k] for k in FIELDS]
            s["groups"] += s["pose_groups"]
        return s
    if kind == "render":
        g, cam, views = _submap(case, seed)
        gs = GaussianSet(**g)
        return dict(kind=kind, batch=_batch(gs, cam, views, None))
    if kind == "register":
        d, P, Q = _pair(case, seed)
        targets = []
        for g, kfs in ((P, d["kf_p"]), (Q, d["kf_q"])):
            imgs = []
            for c in kfs:
                w2c = np.concatenate([c[:3, :3].T, -c[:3, :3].T @ c[:3, 3:4]], 1)
                with torch.no_grad():
                    imgs.append(_render_plain(g, d["cam"], w2c, None, torch.float32))
            targets += [torch.stack([i[0] for i in imgs]).contiguous(), torch.stack([i[1] for i in imgs]).contiguous()]
        args = (GaussianSet(**P), GaussianSet(**Q), d["cam"], d["kf_p"], d["kf_q"], *targets)
        # the learning rates of the paper's synthetic dataset
        return dict(kind=kind, args=args, params=default_params(case["iters"], lr_rot=0.003, lr_trans=0.001))
    if kind == "overlap":
        d, P, Q = _pair(case, seed)
        rng = np.random.default_rng(seed + 1)
        off = synth.pose_matrix4(synth.perturbation(rng, case["rot_deg"], case["trans"]))
        return dict(kind=kind, p=P["mean"], q=Q["mean"], T=off @ d["T_gt"])
    if kind == "prune":
        rng = np.random.default_rng(seed)
        g = synth.gaussians_in_box(rng, case["n"], (-3.0, -1.5, 0.5), (3.0, 1.5, 4.5))
        # the same opacities for every seed, in another order: as many survive
        g["opacity_logit"] = rng.permutation(np.random.default_rng(case["n"]).normal(0.0, 1.0, case["n"]))
        g = _gauss(g)
        gen = torch.Generator(device=DEV).manual_seed(seed)
        extra = [torch.randn(g[k].shape, generator=gen, device=DEV) * 1e-4 for k in FIELDS for _ in range(2)]
        return dict(kind=kind, gs=GaussianSet(**g), extra=extra, threshold=case["threshold"])
    mean, quat, c2w, T = _adjust_inputs(case, seed)
    subs = [(_Submap(case["n"], mean[k], quat[k]), c2w[k] if case["poses"] else None, T[k])
            for k in range(case["submaps"])]
    return dict(kind=kind, subs=subs, mean=mean, quat=quat, c2w=c2w)


class _Submap:
    """What adjust_submaps reads of a submap: its size, means and orientations."""

    def __init__(self, n, mean, quat):
        self.n, self.mean, self.quat = n, mean, quat


def _adjust_inputs(case, seed):
    S, n, k = case["submaps"], case["n"], case["poses"]
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    mean = torch.rand(S, 3, n, generator=gen, device=DEV) * 4.0 - 2.0
    quat = torch.randn(S, 4, n, generator=gen, device=DEV)
    c2w = torch.zeros(S, k, 12, device=DEV)
    c2w[:, :, 0] = c2w[:, :, 5] = c2w[:, :, 10] = 1.0
    c2w[:, :, 3::4] = torch.rand(S, k, 3, generator=gen, device=DEV)
    T = np.stack([synth.pose_matrix4(synth.perturbation(rng, 0.5, 0.01))[:3] for _ in range(S)])
    return mean, quat, c2w, T


# ------------------------------------------------------------------ one pass

def run(s):
    kind = s["kind"]
    b = s.get("batch")
    if kind == "track":
        s["step"] += 1
        b.project(s["pose"])
        b.bin_sort()
        b.render_fwd()
        b.loss_tracking(s["rgb"], s["depth"], loss=s["loss"], median=s["median"], grad_rgb=s["g_rgb"],
                        grad_depth=s["g_depth"], grad_scale=s["scale"])
        b.render_bwd_tiles(s["g_rgb"], s["g_depth"], scale=s["scale"], pose=s["pose"], pose_only=True)
        b.render_bwd_project(pose=s["pose"], pose_grad=s["pose_grad"], pose_only=True)
        adam(s["pose_groups"], s["step"])
        return [b.rgb, b.depth, b.alpha, s["loss"], s["median"], s["g_rgb"], s["g_depth"], s["pose"], s["pm"], s["pv"]]
    if kind == "loop":
        s["step"] += 1
        b.project(s["pose"])
        b.bin_sort()
        b.render_fwd()
        b.render_bwd_tiles_l1(s["rgb"], s["depth"], s["scale"], pose=s["pose"])
        b.loss_l1_tiles(s["loss"])
        b.render_bwd_project_adam([s["moments"]], s["step"], pose=s["pose"], pose_grad=s["pose_grad"],
                                  pose_adam=(s["pm"], s["pv"], LR_ROT, LR_TRANS))
        return [b.rgb, b.depth, b.alpha, s["loss"], s["pose"], s["pm"], s["pv"], s["gs"].tensors(),
                [s["moments"][k][:2] for k in FIELDS]]
    if kind == "map":
        s["step"] += 1
        b.project(s["pose"])
        b.bin_sort()
        b.render_fwd()
        b.loss_mapping(s["rgb"], s["depth"], loss=s["loss"], grad_rgb=s["g_rgb"], grad_depth=s["g_depth"],
                       grad_scale=s["scale"])
        loss_isotropic(s["gs"].log_scale, loss=s["iso"], grad=s["grads"].log_scale, work=s["iso_work"])
        b.render_bwd(s["g_rgb"], s["g_depth"], scale=s["scale"], grads=[s["grads"]], pose=s["pose"],
                     pose_grad=s["pose_grad"])
        adam(s["groups"], s["step"])
        return [b.rgb, b.depth, b.alpha, s["loss"], s["iso"], s["g_rgb"], s["g_depth"], s["pose"], s["pm"], s["pv"],
                s["gs"].tensors(), [s["moments"][k][:2] for k in FIELDS]]
    if kind == "render":
        b.project()
        b.bin_sort()
        b.render_fwd()
        return [b.rgb, b.depth, b.alpha]
    if kind == "grad":
        out = render(b, s["pose"], BG)
        return [t.detach() for t in out], list(torch.autograd.grad(out, s["leaves"], s["up"]))
    if kind == "register":
        r = register_pair(*s["args"], params=s["params"])
        return [np.asarray(r[k], np.float32) for k in ("T", "per_view", "residual")]
    if kind == "overlap":
        return list(overlap_ratio(s["p"], s["q"], s["T"], 0.2))
    if kind == "prune":
        out, kept, extra = prune_gaussians(s["gs"], s["threshold"], s["extra"])
        return [out.tensors(), kept, extra]
    adjust_submaps(s["subs"])
    return [s["mean"], s["quat"], s["c2w"]]


def work(case):
    """Bytes: inputs and outputs once.  Operations: 25 per composited (Gaussian, pixel) forward and 67 with the
    backward, at about 70 per pixel of a full submap (fewer where there are fewer Gaussians than that takes)."""
    kind = case["kind"]
    n = case.get("n", 0)
    pix = case.get("width", 0) * case.get("height", 0)
    if kind in ("track", "loop", "map", "grad"):
        frag = pix * min(70.0, 1.7 * n * (case["focal"] * 0.02 / 2.5 + 0.5) ** 2 * 8 / pix)
        state = dict(track=56, loop=56 + 56 + 4 * 56, map=56 + 56 + 4 * 56, grad=2 * 56)[kind]
        return dict(bytes=state * n + dict(track=52, loop=36, map=52, grad=40)[kind] * pix,
                    flops=67 * frag + (3 * 390 * pix if kind == "map" else 0))
    if kind == "render":
        return dict(bytes=56 * n + 20 * pix * case["views"], flops=25 * 40.0 * pix * case["views"])
    if kind == "register":
        v = case["views"]
        frag = 40.0 * pix * 2 * v
        return dict(bytes=case["iters"] * (56 * v * (case["n_p"] + case["n_q"]) + 32 * pix * v),
                    flops=case["iters"] * 67 * frag)
    if kind == "overlap":
        m = case["n_p"] + case["n_q"]
        return dict(bytes=16 * m, flops=8.0 * 128 * m)
    if kind == "prune":
        return dict(bytes=4 * n * 42 + 4 * (n // 2) * 43, flops=n)
    return dict(bytes=case["submaps"] * (56 * n + 96 * case["poses"]), flops=46.0 * n * case["submaps"])


# ------------------------------------------------------------------ plain PyTorch, for measurements and exact values

def _rot(q):
    w, x, y, z = (q / q.norm(dim=0, keepdim=True)).unbind(0)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)])


def _project_plain(g, cam, w2c, pose):
    """Splat centres, conics and depths, and the FP32 decisions that the lists rest on: radius and tiles."""
    A = torch.as_tensor(np.asarray(w2c, np.float32), device=DEV).to(g["mean"].dtype)
    R, t = A[:, :3], A[:, 3]
    if pose is not None:
        Rd = _rot(pose[:4, None]).view(3, 3)
        R, t = (Rd[:, :, None] * R[None]).sum(1), (Rd * t).sum(1) + pose[4:]
    p = [sum(R[i, k] * g["mean"][k] for k in range(3)) + t[i] for i in range(3)]
    Rq, sc = _rot(g["quat"]), g["log_scale"].exp()
    V = [[sum(R[i, k] * Rq[3 * k + j] for k in range(3)) * sc[j] for j in range(3)] for i in range(3)]
    x, y, z = p
    U0 = [cam["fx"] / z * V[0][j] - cam["fx"] * x / (z * z) * V[2][j] for j in range(3)]
    U1 = [cam["fy"] / z * V[1][j] - cam["fy"] * y / (z * z) * V[2][j] for j in range(3)]
    a = sum(u * u for u in U0) + 0.3
    b = sum(u * v for u, v in zip(U0, U1))
    c = sum(u * u for u in U1) + 0.3
    det = a * c - b * b
    u, v = cam["fx"] * x / z + cam["cx"], cam["fy"] * y / z + cam["cy"]
    with torch.no_grad():
        a3, b3, c3, u3, v3, z3 = (k.float() for k in (a, b, c, u, v, z))
        h = 0.5 * (a3 - c3)
        rad = torch.ceil(3.0 * torch.sqrt(0.5 * (a3 + c3) + torch.sqrt(h * h + b3 * b3)))
        rad = torch.where((z3 > 0.2) & (a3 * c3 - b3 * b3 > 0), rad, torch.zeros_like(rad))
        tx, ty = (cam["width"] + 15) // 16, (cam["height"] + 15) // 16
        x0, x1 = (torch.floor((u3 - rad) / 16).clamp(0, tx), (torch.floor((u3 + rad) / 16) + 1).clamp(0, tx))
        y0, y1 = (torch.floor((v3 - rad) / 16).clamp(0, ty), (torch.floor((v3 + rad) / 16) + 1).clamp(0, ty))
        cnt = torch.where(rad > 0, (x1 - x0).clamp(min=0) * (y1 - y0).clamp(min=0), torch.zeros_like(rad)).long()
        kept = cnt.nonzero().flatten()
        kept = kept[torch.sort(z3[kept], stable=True).indices]
        rep = kept.repeat_interleave(cnt[kept])
        first = torch.cumsum(cnt[kept], 0) - cnt[kept]
        q = torch.arange(rep.numel(), device=DEV) - first.repeat_interleave(cnt[kept])
        wid = (x1 - x0).long()[rep]
        tile = (y0.long()[rep] + q // wid) * tx + x0.long()[rep] + q % wid
        order = torch.sort(tile, stable=True).indices
        lists = rep[order], torch.bincount(tile, minlength=tx * ty)
    return dict(u=u, v=v, ca=c / det, cb=-b / det, cc=a / det, z=z), lists


def _composite_tiles(s, ids, valid, px, py):
    """Front-to-back compositing of tiles with equally long lists: [4, pixels] colour and depth, transmittance."""
    dx, dy = px[:, None] - s["u"][ids][..., None], py[:, None] - s["v"][ids][..., None]
    sig = 0.5 * (s["ca"][ids][..., None] * dx * dx + s["cc"][ids][..., None] * dy * dy) \
        + s["cb"][ids][..., None] * dx * dy
    al = (s["o"][ids][..., None] * torch.exp(-sig)).clamp(max=float(np.float32(0.99)))
    hit = (sig >= 0) & (al >= float(np.float32(1 / 255))) & valid[..., None]
    al = torch.where(hit, al, torch.zeros_like(al))
    after = torch.cumprod(1 - al, 1)
    live = torch.cumsum(hit & (after.detach() < float(np.float32(1e-4))), 1) == 0
    before = torch.cat([torch.ones_like(after[:, :1]), after[:, :-1]], 1)
    w = al * before * live
    T = torch.where(live, after, torch.ones_like(after)).amin(1)
    return torch.stack([(w * s["col"][k][ids][..., None]).sum(1) for k in range(4)], 1), T


def _splat(g, cam, w2c, pose, dtype):
    g = {k: v.to(dtype) for k, v in g.items()}
    s, lists = _project_plain(g, cam, w2c, None if pose is None else pose.to(dtype))
    s["o"] = torch.sigmoid(g["opacity_logit"])
    s["col"] = torch.cat([g["rgb"], s["z"][None]])
    return s, lists


def _tile_groups(lists, cam):
    """Tiles in groups of about equal list length, with their padded lists and pixels."""
    items, count = lists
    start = torch.cumsum(count, 0) - count
    order = torch.sort(count, descending=True, stable=True).indices
    sorted_count = count[order].tolist()
    tx = (cam["width"] + 15) // 16
    i = 0
    while i < len(sorted_count) and sorted_count[i] > 0:
        k = sorted_count[i]
        t = order[i:i + max(1, 20_000_000 // (256 * k))]
        t = t[count[t] > 0]
        at = torch.arange(k, device=DEV)
        valid = at[None] < count[t][:, None]
        ids = items[(start[t][:, None] + at[None]).clamp(max=items.numel() - 1)]
        sub = torch.arange(256, device=DEV)
        x, y = (t % tx)[:, None] * 16 + sub % 16, (t // tx)[:, None] * 16 + sub // 16
        yield ids, valid, x, y
        i += t.numel()


def _render_plain(g, cam, w2c, pose, dtype, bg=None):
    """(rgb [3, H, W], depth, alpha [H, W]) in `dtype`, without this package's kernels."""
    s, lists = _splat(g, cam, w2c, pose, dtype)
    return _images(s, lists, cam, dtype, bg)


def _images(s, lists, cam, dtype, bg):
    W, H = cam["width"], cam["height"]
    img = torch.zeros(4, H * W, dtype=dtype, device=DEV)
    T = torch.ones(H * W, dtype=dtype, device=DEV)
    for ids, valid, x, y in _tile_groups(lists, cam):
        c, t = _composite_tiles(s, ids, valid, x.to(dtype) + 0.5, y.to(dtype) + 0.5)
        inside = (x < W) & (y < H)
        p = (y * W + x)[inside]
        img[:, p] = c.permute(1, 0, 2)[:, inside]
        T[p] = t[inside]
    bg = torch.tensor([0.0, 0.0, 0.0] if bg is None else [float(np.float32(v)) for v in bg], dtype=dtype, device=DEV)
    return (img[:3] + T * bg[:, None]).view(3, H, W), img[3].view(H, W), (1 - T).view(H, W)


def _exact_grads(g, cam, w2c, pose, bg, upstream):
    """64-bit images, and the gradients of pose and Gaussians under upstream(rgb, depth, alpha)."""
    leaves = {k: v.double().requires_grad_(True) for k, v in g.items()}
    pose = pose.double().requires_grad_(True)
    s, lists = _splat(leaves, cam, w2c, pose, torch.float64)
    cut = {k: v.detach().requires_grad_(True) for k, v in s.items()}
    with torch.no_grad():
        img = _images(cut, lists, cam, torch.float64, bg)
    extra, (g_rgb, g_depth, g_alpha) = upstream(*img)
    W, H = cam["width"], cam["height"]
    g4 = torch.cat([g_rgb.view(3, -1), g_depth.view(1, -1)])
    g_T = -g_alpha.reshape(-1)
    if bg is not None:
        g_T = g_T + sum(float(np.float32(bg[k])) * g4[k] for k in range(3))
    for ids, valid, x, y in _tile_groups(lists, cam):
        inside = (x < W) & (y < H)
        p = torch.where(inside, y * W + x, torch.zeros_like(x))
        m = inside.double()
        c, t = _composite_tiles(cut, ids, valid, x.double() + 0.5, y.double() + 0.5)
        torch.autograd.backward([c, t], [g4[:, p].permute(1, 0, 2) * m[:, None], g_T[p] * m])
    names = [k for k in s if cut[k].grad is not None]
    torch.autograd.backward([s[k] for k in names], [cut[k].grad for k in names])
    grads = {k: v.grad if v.grad is not None else torch.zeros_like(v) for k, v in leaves.items()}
    return img, extra, (g_rgb, g_depth), grads, pose.grad


def _l1(tgt, tgt_d):
    def up(rgb, depth, alpha):
        ok = (tgt_d > 0).double()
        inv = 1.0 / ok.sum()
        loss = ((rgb - tgt).abs().sum(0) + (depth - tgt_d).abs()).mul(ok).sum() * inv
        return loss, (torch.sign(rgb - tgt) * ok * inv, torch.sign(depth - tgt_d) * ok * inv, torch.zeros_like(depth))
    return up


def _tracking(tgt, tgt_d, lc=float(np.float32(0.6)), k=50.0):
    def up(rgb, depth, alpha):
        ok = tgt_d > 0
        e = (depth - tgt_d).abs()
        med = e[ok].kthvalue((int(ok.sum()) - 1) // 2 + 1).values
        w = (ok & (e <= k * med)).double() * alpha ** 3
        inv = 1.0 / ok.double().sum()
        loss = (w * (lc * (rgb - tgt).abs().sum(0) + (1 - lc) * e)).sum() * inv
        g_rgb, g_d = w * lc * torch.sign(rgb - tgt), w * (1 - lc) * torch.sign(depth - tgt_d)
        return (loss, med, g_rgb, g_d), (g_rgb * inv, g_d * inv, torch.zeros_like(depth))
    return up


def _mapping(tgt, tgt_d, ls=float(np.float32(0.2))):
    k = torch.arange(11, dtype=torch.float64, device=DEV) - 5
    win = torch.exp(-k * k / 4.5)
    win = win / win.sum()

    def blur(x):
        H, W = x.shape[-2:]
        x = torch.nn.functional.pad(x, (5, 5, 5, 5))
        x = sum(win[i] * x[..., i:i + W] for i in range(11))
        return sum(win[i] * x[..., i:i + H, :] for i in range(11))

    def up(rgb, depth, alpha):
        rgb, depth = rgb.clone().requires_grad_(True), depth.clone().requires_grad_(True)
        ok = (tgt_d > 0).double()
        mx, my = blur(rgb), blur(tgt)
        vx, vy, cxy = blur(rgb * rgb) - mx * mx, blur(tgt * tgt) - my * my, blur(rgb * tgt) - mx * my
        ssim = (2 * mx * my + 1e-4) * (2 * cxy + 9e-4) / ((mx * mx + my * my + 1e-4) * (vx + vy + 9e-4))
        l1 = ((rgb - tgt).abs().sum(0) * ok).sum() / ok.sum()
        loss = (1 - ls) * l1 + ls * (1 - ssim.mean()) + ((depth - tgt_d).abs() * ok).sum() / ok.sum()
        g_rgb, g_d = torch.autograd.grad(loss, [rgb, depth])
        return loss.detach(), (g_rgb, g_d, torch.zeros_like(depth))
    return up


def _adam_exact(p, grad, m, v, lr, step, b1=float(np.float32(0.9)), b2=float(np.float32(0.999))):
    p, m, v = p.double(), m.double(), v.double()
    m = b1 * m + (1 - b1) * grad
    v = b2 * v + (1 - b2) * grad * grad
    return p - lr * (m / (1 - b1 ** step)) / ((v / (1 - b2 ** step)).sqrt() + 1e-8), m, v


def exact(case, seed):
    kind = case["kind"]
    if kind in ("track", "loop", "map", "grad"):
        g, cam, w2c, rgb, depth = _volume(case, seed)
        pose, _, pm, pv = _pose_state(seed)
        up = dict(track=_tracking, loop=_l1, map=_mapping, grad=lambda *a: None)[kind](rgb.double(), depth.double())
        if kind == "grad":
            gen = torch.Generator(device=DEV).manual_seed(seed + 9)
            npix = case["width"] * case["height"]
            u = [(torch.randn(k * npix, generator=gen, device=DEV) / npix).double() for k in (3, 1, 1)]

            def up(r, d, a):
                return None, (u[0].view_as(r), u[1].view_as(d), u[2].view_as(a))
        img, extra, g_img, grads, g_pose = _exact_grads(g, cam, w2c, pose[0], BG if kind == "grad" else None, up)
        img = [t.reshape(-1) for t in img]
        if kind == "grad":
            return img, [g_pose[None]] + [grads[k] for k in FIELDS]
        step = STEP0 + 1
        q = _adam_exact(pose[:, :4], g_pose[None, :4], pm[:, :4], pv[:, :4], LR_ROT, step)
        t = _adam_exact(pose[:, 4:], g_pose[None, 4:], pm[:, 4:], pv[:, 4:], LR_TRANS, step)
        pose_out = [torch.cat([a, b], 1) for a, b in zip(q, t)]
        if kind == "track":
            loss, med, g_rgb, g_d = extra
            return img + [loss[None], med[None], g_rgb.reshape(-1), g_d.reshape(-1)] + pose_out
        iso = None
        if kind == "map":
            ls = g["log_scale"].double().requires_grad_(True)
            sc = ls.exp()
            iso = (sc - sc.mean(0)).abs().sum() / case["n"]
            grads["log_scale"] = grads["log_scale"] + torch.autograd.grad(iso, ls)[0]
        mom = _moments(g, case, seed)
        new = [_adam_exact(g[k], grads[k], *mom[k], step) for k in FIELDS]
        tail = pose_out + [[a[0] for a in new], [a[1:] for a in new]]
        if kind == "loop":
            return img + [extra[None]] + tail
        return img + [extra[None], iso.detach()[None], g_img[0].reshape(-1), g_img[1].reshape(-1)] + tail
    if kind == "render":
        g, cam, views = _submap(case, seed)
        with torch.no_grad():
            imgs = [_render_plain(g, cam, w, None, torch.float64) for w in views]
        return [torch.cat([i[k].reshape(-1) for i in imgs]) for k in range(3)]
    if kind == "register":
        return None  # tens of renders, and every step's rounding travels through the rest
    if kind == "overlap":
        s = prepare(case, seed)
        T = torch.as_tensor(s["T"][:3].astype(np.float32), device=DEV).double()
        p = [sum(T[r, k] * s["p"][k].double() for k in range(3)) + T[r, 3] for r in range(3)]
        q = [s["q"][k].double() for k in range(3)]
        near, back, close = [], torch.full_like(q[0], math.inf), torch.zeros(q[0].numel(), dtype=torch.long, device=DEV)
        dist = []
        for i in range(0, p[0].numel(), 1024):
            d2 = sum((p[k][i:i + 1024, None] - q[k][None]) ** 2 for k in range(3))
            m = d2.min(1)
            near.append(m.indices)
            dist.append(m.values)
            m = d2.min(0)
            better = m.values < back
            back, close = torch.where(better, m.values, back), torch.where(better, m.indices + i, close)
        near, dist = torch.cat(near), torch.cat(dist)
        pair = close[near] == torch.arange(near.numel(), device=DEV)
        return [float((pair & (dist < float(np.float32(0.2)) ** 2)).sum()) / max(1, int(pair.sum())), None, None, None,
                None]
    if kind == "prune":
        s = prepare(case, seed)
        keep = s["gs"].opacity_logit >= np.float32(math.log(case["threshold"] / (1 - case["threshold"])))
        return [[t.double()[..., keep] for t in s["gs"].tensors()], None, [t.double()[..., keep] for t in s["extra"]]]
    mean, quat, c2w, T = _adjust_inputs(case, seed)
    T = torch.as_tensor(T.astype(np.float32), device=DEV).double()
    R, t = T[:, :, :3], T[:, :, 3]
    out_mean = sum(R[:, :, k:k + 1] * mean[:, k:k + 1].double() for k in range(3)) + t[:, :, None]
    w1 = 0.5 * (1 + R[:, 0, 0] + R[:, 1, 1] + R[:, 2, 2]).sqrt()
    x1, y1, z1 = ((R[:, i, j] - R[:, j, i]) / (4 * w1) for i, j in ((2, 1), (0, 2), (1, 0)))
    qn = (w1 * w1 + x1 * x1 + y1 * y1 + z1 * z1).sqrt()
    w1, x1, y1, z1 = ((k / qn)[:, None] for k in (w1, x1, y1, z1))
    w, x, y, z = quat.double().unbind(1)
    out_quat = torch.stack([w1 * w - x1 * x - y1 * y - z1 * z, w1 * x + x1 * w + y1 * z - z1 * y,
                            w1 * y - x1 * z + y1 * w + z1 * x, w1 * z + x1 * y - y1 * x + z1 * w], 1)
    P = c2w.double().view(c2w.shape[0], c2w.shape[1], 3, 4)
    out_c2w = sum(R[:, None, :, k, None] * P[:, :, k, None, :] for k in range(3))
    out_c2w[..., 3] += t[:, None]
    return [out_mean, out_quat, out_c2w.reshape(c2w.shape)]
