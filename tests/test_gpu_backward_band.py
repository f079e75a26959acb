"""The band-wise compositing backward at the edges of its batches: lists whose
composited entries fill a group of eight, a staged batch of 32, a word of 64
"used" bits or 64 such words exactly, fall one short or go one over, on an
image that cuts tiles and bands."""

import math

import numpy as np
import pytest
import torch

from tests import _util as U

pytestmark = pytest.mark.gpu


def _scene(n, seed):
    """n small, faint Gaussians over the first tile of a 20 x 13 image, few
    enough per pixel that compositing never stops early."""
    from paper_2408_10154_amd import synth

    rng = np.random.default_rng(seed)
    g = synth.gaussians_in_box(rng, n, (-1, -1, 0), (1, 1, 1))
    z = rng.uniform(1.5, 3.0, n)
    u, v = rng.uniform(3.0, 13.0, n), rng.uniform(1.0, 12.0, n)
    g["mean"] = np.stack([(u - 10.0) / 20.0 * z, (v - 6.5) / 20.0 * z, z]).astype(np.float32)
    g["log_scale"] = (np.log(1.2 / 20.0 * z) + rng.normal(0, 0.1, (3, n))).astype(np.float32)
    o = 0.012 if n > 500 else 0.3
    g["opacity_logit"] = np.full(n, math.log(o / (1 - o)), np.float32) + rng.normal(0, 0.05, n).astype(np.float32)
    return g, synth.camera(20, 20, 10, 6.5, 20, 13), synth.identity_w2c(), synth.perturbation(rng, 1.0, 0.01)


@pytest.mark.parametrize("n", [1, 7, 8, 9, 31, 32, 33, 63, 64, 65, 130, 4200])
def test_backward_at_batch_edges(gpu, n):
    """Gradients of a random linear function of the images to the Gaussians
    and the pose (full and pose-only) within 1e-3 of the oracle in norm: FP32
    sums over at most 256 pixels and a few hundred entries, and decisions
    within rounding of their thresholds, which move an image by < 1/255."""
    from paper_2408_10154_amd.render import GaussianSet, RenderBatch

    g, cam, w2c, pose = _scene(n, n)
    b = RenderBatch([(GaussianSet.from_numpy(g), cam, w2c)])
    pt = torch.as_tensor(pose[None], device="cuda")
    b.project(pt)
    b.bin_sort()
    b.render_fwd()
    P = b.P
    rng = np.random.default_rng(1)
    up = [rng.normal(size=s).astype(np.float32) for s in (3 * P, P, P)]
    upd = [torch.as_tensor(u, device="cuda") for u in up]
    grads, pg = [b.gsets[0].zeros_like()], torch.zeros_like(pt)
    b.render_bwd(*upd, grads=grads, pose=pt, pose_grad=pg)
    pg_only = torch.zeros_like(pt)
    b.render_bwd_tiles(*upd, pose=pt, pose_only=True)
    b.render_bwd_project(pose=pt, pose_grad=pg_only, pose_only=True)
    torch.cuda.synchronize()

    gt, ptt, o = U.oracle_render(g, cam, w2c, pose, requires_grad=True)
    H, W = cam["height"], cam["width"]
    ur, ud, ua = (torch.as_tensor(u, dtype=torch.float64) for u in up)
    ((o["rgb"] * ur.view(3, H, W)).sum() + (o["depth"] * ud.view(H, W)).sum() +
     (o["alpha"] * ua.view(H, W)).sum()).backward()
    if n == 4200:
        assert int(b.n_last.max()) > 4096, "the list must outgrow 64 words of used bits"
    for name in ("mean", "log_scale", "quat", "opacity_logit", "rgb"):
        got = getattr(grads[0], name).cpu().numpy()
        err = U.rel_err(got.T if got.ndim == 2 else got, gt[name].grad.numpy())
        assert err < 1e-3, (n, name, err)
    for got in (pg, pg_only):
        err = U.rel_err(got[0].cpu().numpy(), ptt.grad.numpy())
        assert err < 1e-3, (n, "pose", err)
