"""The adjoint voxel pass where its workgroups differ: views split over several
workgroups of a small grid, workgroups all of whose voxels scatter (labels at
odds with the images) or none (most, with the true labels), boxes staged in
groups of views and boxes that fit no group. Gradients against the FP64 oracle
at the tolerance of the other differentiable tests: fixed-point terms are
rounded to 2^-20 of the largest, of which a pixel that matters sums many."""
import numpy as np
import pytest

from oracle import oracle as O
from synth import scene as S
from tests.test_parity_diff import check_grads, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,n,f,W,H,labels,sub", [
    ((17, 9, 9), 16, 150.0, 161, 119, "random", None),            # one view per workgroup
    ((33, 16, 8), 5, 150.0, 161, 119, "random", [16, 33, 0, 16, 0, 8]),   # workgroups outside the region
    ((40, 48, 33), 7, 190.0, 203, 151, "true", None),             # ragged, views split unevenly
    ((64, 64, 64), 12, 150.0, 161, 119, "true", None),            # several groups, most workgroups cold
    ((48, 40, 56), 4, 900.0, 640, 480, "true", None),             # boxes that fit no group
])
def test_gradients_follow_the_oracle(dims, n, f, W, H, labels, sub):
    rng = np.random.default_rng(dims[0] * 100 + n)
    cams = S.perturb_cameras(S.ring_rig(n, f, W, H), seed=(20, n), rel=0.002)
    voxel = np.float32(2.0 / max(dims))
    grid = S.Grid(*dims, np.array([-0.5 * voxel * d for d in dims], np.float32), voxel)
    body = S.make_body(rng)
    fr = S.render_frame(20, n, cams, grid, body, (20, n))
    lab = S.gt_occupancy(grid, body) if labels == "true" else (rng.random(dims[::-1]) < 0.5).astype(np.uint8)
    logits, loss, gm, gv, gP = run_gpu(fr, cams, lab, sub, grad_loss=1.7)
    ref = O.grad(cams, grid, fr.images, fr.mean, fr.var, lab, sub, grad_loss=1.7)
    check_grads(gm, gv, gP, ref, f"{dims} x {n}")
