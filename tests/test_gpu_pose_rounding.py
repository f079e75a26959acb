"""The pose-only gradient and the registrations that follow it, bit for bit.

A registration takes tens to hundreds of Adam steps along its pose gradients, and
Adam's quotient turns a changed last bit of a component that cancels into
another pose: views' residuals move by up to 1e-4 of themselves with the order in
which a gradient is summed.  So the gradient's rounding is part of what a
registration returns.  tests/golden/pose_gradients.json holds the values (as FP32
bit patterns) of the tile-wise backward that the registrations of earlier
releases were computed with, on the scenes below."""

import json
import math
import os

import numpy as np
import pytest
import torch

from paper_2408_10154_amd import synth

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "pose_gradients.json")

# (one tile with every entry at every pixel it covers, or spread over the image), image, items, opacity: list lengths
# around chunks of 64 positions and rounds of 128 and 256, few and more than 128 composited entries in a round
SCENES = [("heap", 16, 16, n, o) for n, o in ((1, 0.05), (2, 0.995), (9, 0.05), (64, 0.05), (65, 0.3), (128, 0.02),
                                              (129, 0.02), (256, 0.02), (257, 0.02), (300, 0.012), (1500, 0.012))]
SCENES += [("spread", w, h, n, o) for w, h, n, o in ((16, 16, 30, 0.995), (16, 16, 1500, 0.02), (8, 8, 257, 0.05),
                                                     (13, 21, 130, 0.3), (64, 48, 600, 0.05), (64, 48, 4000, 0.3))]
PAIRS = [(1, "l1"), (2, "l1"), (3, "tracking")]


def pose_gradients(kind, W, H, n, o):
    """Pose gradients of random linear functions of the colour, of the depth and of all images."""
    from paper_2408_10154_amd.render import GaussianSet, RenderBatch

    rng = np.random.default_rng(1000 * n + W)
    g = synth.gaussians_in_box(rng, n, (-1, -1, 0), (1, 1, 1))
    z = rng.uniform(1.5, 3.0, n)
    lo, hi = ((3, 3), (5, 5)) if kind == "heap" else ((0, 0), (W, H))
    u, v = (rng.uniform(lo[k], hi[k], n) for k in range(2))
    g["mean"] = np.stack([(u - W / 2) / 20.0 * z, (v - H / 2) / 20.0 * z, z]).astype(np.float32)
    g["log_scale"] = (np.log(1.2 / 20.0 * z) + rng.normal(0, 0.3, (3, n))).astype(np.float32)
    g["opacity_logit"] = (math.log(o / (1 - o)) + rng.normal(0, 0.05, n)).astype(np.float32)
    b = RenderBatch([(GaussianSet.from_numpy(g), synth.camera(20, 20, W / 2, H / 2, W, H), synth.identity_w2c())])
    pose = torch.as_tensor(synth.perturbation(rng, 1.0, 0.01)[None], device="cuda")
    b.project(pose)
    b.bin_sort()
    b.render_fwd()
    up = [torch.as_tensor(rng.normal(size=s).astype(np.float32), device="cuda") for s in (3 * b.P, b.P, b.P)]
    out = []
    for a in ((up[0], None, None), (None, up[1], None), up):
        grad = torch.zeros_like(pose)
        b.render_bwd_tiles(*a, pose=pose, pose_only=True)
        b.render_bwd_project(pose=pose, pose_grad=grad, pose_only=True)
        out.append(grad.cpu().numpy())
    return np.concatenate(out)


def registration(seed, loss):
    """Transform, per-view estimates and residuals of a small pair."""
    from paper_2408_10154_amd import register as REG
    from paper_2408_10154_amd.render import GaussianSet

    d = synth.registration_pair(seed, 3000, 2500, shared_frac=0.9, views_p=2, views_q=3, width=150, height=110, f=100,
                                half=(1.0, 0.6, 0.8), log_scale_mu=math.log(0.05), rot_deg_max=2.0, trans_max=0.03)
    P, Q = GaussianSet.from_numpy(d["P"]), GaussianSet.from_numpy(d["Q"])
    targets = (*REG.keyframe_targets(P, d["cam"], d["kf_p"]), *REG.keyframe_targets(Q, d["cam"], d["kf_q"]))
    params = REG.default_params(20, 0.003, 0.001, loss=loss)
    r = REG.register_pair(P, Q, d["cam"], d["kf_p"], d["kf_q"], *targets, params)
    return np.concatenate([np.asarray(r[k], np.float32).reshape(-1) for k in ("T", "per_view", "residual")])


def _equal(got, key):
    with open(GOLDEN) as f:
        want = np.array(json.load(f)[key], np.uint32).view(np.float32).reshape(got.shape)
    np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("scene", SCENES, ids=str)
def test_pose_gradient_bits(gpu, scene):
    _equal(pose_gradients(*scene), str(scene))


@pytest.mark.parametrize("pair", PAIRS, ids=str)
def test_registration_bits(gpu, pair):
    _equal(registration(*pair), str(pair))
