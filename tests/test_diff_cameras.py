"""occupancy_loss with camera matrices on the GPU: a plan's later calls read
them beside the likelihood maps (psfs_diff_forward_at); every result has the
bits of the first call's separate steps, and what those refuse is refused."""
import numpy as np
import pytest
import torch

import paper_1311_6811_amd as psfs
from paper_1311_6811_amd import _lib as L
from gpu_util import upload
from synth import scene as S


def _scene(n):
    fr = S.config_frame(0, 1)
    ims, mus, vs = upload(fr)
    labels = torch.from_numpy(S.gt_occupancy(fr.grid, fr.body)).cuda()
    P = torch.tensor(np.stack([c.P for c in S.perturb_cameras(fr.cams, seed=(4, 1))][:n]).reshape(n, 3, 4), dtype=torch.float32)
    return fr, ims[:n], [m.requires_grad_(True) for m in mus[:n]], [v.requires_grad_(True) for v in vs[:n]], labels, P


def _grads(P, mus, vs, ims, labels, plan):
    P = P.detach().requires_grad_(True)
    loss = psfs.occupancy_loss(P, mus, vs, ims, labels, plan)
    return [loss.detach(), *torch.autograd.grad(loss, [P, *mus, *vs])]


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 4])
def test_later_calls_repeat_the_first(n):
    fr, ims, mus, vs, labels, P = _scene(n)
    first = _grads(P, mus, vs, ims, labels, psfs.DiffPlan(fr.cams[:n], fr.grid))     # host matrices
    plan = psfs.DiffPlan(fr.cams[:n], fr.grid)
    _grads((P + 1.0).cuda(), mus, vs, ims, labels, plan)
    wide = torch.zeros((n, 3, 8), device="cuda")
    wide[..., ::2] = P.cuda()
    for Q in (P.cuda(), P.cuda().double(), wide[..., ::2]):
        again = _grads(Q, mus, vs, ims, labels, plan)
        for a, b in zip(first, again):
            assert torch.equal(a.cpu(), b.to("cpu", a.dtype))
    assert np.array_equal(np.stack([np.asarray(c.P).reshape(3, 4) for c in plan.cams]), P.numpy())


@pytest.mark.gpu
def test_refusals_leave_the_plan_usable():
    fr, ims, mus, vs, labels, P = _scene(4)
    plan = psfs.DiffPlan(fr.cams, fr.grid)
    good = _grads(P.cuda(), mus, vs, ims, labels, plan)
    bad = P.clone()
    bad[2, 1, 3] = float("nan")
    for Q in (bad, bad.cuda()):
        with pytest.raises(psfs.PsfsError, match="view 2: camera matrix not finite"):
            _grads(Q, mus, vs, ims, labels, plan)
    with pytest.raises(IndexError):
        _grads(P[:3].cuda(), mus[:3], vs[:3], ims[:3], labels, plan)
    with pytest.raises(psfs.PsfsError, match="background of view 3"):
        psfs.occupancy_loss(P.cuda(), mus, vs[:3], ims, labels, plan)
    with pytest.raises(TypeError):
        psfs.occupancy_loss(P.cuda(), mus, [*vs[:3], vs[3].cpu()], ims, labels, plan)
    for a, b in zip(good, _grads(P.cuda(), mus, vs, ims, labels, plan)):
        assert torch.equal(a, b)


def test_set_views_refuses_before_it_sets():
    lib = L.lib()
    plan = psfs.Plan([S.config_frame(0, 0).cams[0]])
    cam = psfs.api.make_camera(8, 6, np.eye(3, 4))
    arr, bg, odd = (L.psfs_camera * 1)(cam), L.ptr_array([256]), L.ptr_array([260])
    size = plan.lmap_floats()
    assert lib.psfs_set_views(plan.handle, 1, arr, None, bg) == -1
    assert lib.psfs_set_views(plan.handle, 1, arr, bg, odd) == -1
    assert lib.psfs_set_views(plan.handle, 17, arr, bg, bg) == -2
    assert lib.psfs_set_views(None, 1, arr, bg, bg) == -1
    assert plan.lmap_floats() == size
    assert lib.psfs_set_views(plan.handle, 1, arr, bg, bg) == 0
    assert plan.lmap_floats() == 64
    assert lib.psfs_diff_forward_at(plan.handle, 2, arr, 256, bg, bg, bg, None, None, None, None, None, 0, None) == -1
