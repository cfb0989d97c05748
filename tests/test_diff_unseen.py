"""The differentiable pass where its views differ: some seen through pixel boxes, some
from among the voxels (no box), some out of sight of part of the grid or of all of it,
in turn, in workgroups all of whose voxels scatter (labels at odds with the images) and in
those with none. Logits and gradients against the FP64 oracle at the tolerances of
the other differentiable tests; a view that sees no voxel gets gradients of 0."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import scene as S
from tests.test_parity_diff import LOGIT_TOL, check_grads, run_gpu

pytestmark = pytest.mark.gpu


def _views(n, f, W, H):
    """Every view in turn as it is, among the voxels, and shifted half out of the image."""
    half = np.array([[1.0, 0.0, 0.55 * W], [0.0, 1.0, 0.0], [0.0, 0.0, 1.0]])
    rings = [S.ring_rig(n, f, W, H), S.ring_rig(n, f, W, H, 0.4, 0.2), S.ring_rig(n, f, W, H, 2.2)]
    cams = [rings[k % 3][k] for k in range(n)]
    return [c.with_P(half @ c.P) if k % 3 == 2 else c for k, c in enumerate(cams)]


@pytest.mark.parametrize("dims,n,labels", [
    ((40, 48, 33), 7, "random"),
    ((40, 48, 33), 7, "true"),
    ((96, 96, 66), 3, "true"),                  # few views: not split
    ((81, 83, 130), 12, "true"),                # many views of 612 blocks: split
])
def test_views_of_every_kind_follow_the_oracle(dims, n, labels):
    rng = np.random.default_rng(dims[0] * 100 + n)
    cams = S.perturb_cameras(_views(n, 150.0, 161, 119), seed=(21, n), rel=0.002)
    gone = n - 1                                # the last view looks past the whole grid
    cams[gone] = cams[gone].with_P(np.array([[1.0, 0.0, 1e5], [0.0, 1.0, 0.0], [0.0, 0.0, 1.0]]) @ S.ring_rig(n, 150.0, 161, 119)[gone].P)
    voxel = np.float32(2.0 / max(dims))
    grid = S.Grid(*dims, np.array([-0.5 * voxel * d for d in dims], np.float32), voxel)
    body = S.make_body(rng)
    fr = S.render_frame(21, n, cams, grid, body, (21, n))
    lab = S.gt_occupancy(grid, body) if labels == "true" else (rng.random(dims[::-1]) < 0.5).astype(np.uint8)
    logits, loss, gm, gv, gP = run_gpu(fr, cams, lab, None, grad_loss=1.7)
    ref = O.grad(cams, grid, fr.images, fr.mean, fr.var, lab, None, grad_loss=1.7)
    check_grads(gm[:gone], gv[:gone], gP[:gone], [r[:gone] for r in ref], f"{dims} x {n}")
    L = O.bilinear_logits(cams, grid, [O.log2slm(i, m, v) for i, m, v in zip(fr.images, fr.mean, fr.var)])
    assert float(np.max(np.abs(logits.astype(np.float64) - L))) <= LOGIT_TOL
    for g in (gm[gone], gv[gone], gP[gone]):
        assert not np.asarray(g).any()
