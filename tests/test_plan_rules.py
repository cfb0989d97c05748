"""A plan's tile and its views that hold the grid follow the settings, whichever
of them changes between two calls: the reported tile, and the bits of a plan
that was made for the settings."""
import numpy as np
import pytest
import torch

import paper_1311_6811_amd as psfs
from synth import scene as S


class _Grid:
    def __init__(self, n, side):
        self.nx = self.ny = self.nz = n
        self.voxel = np.float32(side / n)
        self.origin = np.full(3, -0.5 * n * self.voxel, np.float32)


def _cams(radius=4.0):
    return S.ring_rig(6, 300.0, 320, 240, radius)


def test_the_tile_follows_every_setting():
    plan = psfs.Plan(_cams(), _Grid(40, 2.0))
    assert plan.tile == 3 == plan.tile
    plan.set_grid(_Grid(112, 2.0))
    assert plan.tile == 2
    plan.set_params(sampling=psfs.BILINEAR)
    assert plan.tile == 6
    plan.set_cameras(S.ring_rig(6, 3000.0, 3200, 2400))
    assert plan.tile == 0
    plan.set_params()
    assert plan.tile == 2
    plan.set_grid(_Grid(40, 2.0))
    assert plan.tile == 3


@pytest.mark.gpu
@pytest.mark.parametrize("sampling", [psfs.NEAREST, psfs.BILINEAR])
def test_every_setting_between_two_calls(sampling):
    plan = psfs.Plan(_cams(), _Grid(50, 1.0), sampling=sampling)
    lmap = torch.empty(plan.lmap_floats(), device="cuda").uniform_(-6.0, 0.6)
    maps2, maps4 = lmap.repeat_interleave(2), lmap.repeat_interleave(4)

    def outputs(p):
        post, occ = p.fuse(lmap)
        step = torch.empty_like(post)
        p.pipeline_step(None, None, lmap, step)
        out = [post, occ, step]
        if p.params.sampling == psfs.NEAREST:
            more = [torch.empty_like(post) for _ in range(6)]
            p.pipeline_step_pair(None, None, None, maps2, more[0], None, more[1], None)
            p.pipeline_step_quad(None, None, maps4, more[2:], None)
            out += more
        return out

    def check(cams, grid, sampling):
        fresh = psfs.Plan(cams, grid, sampling=sampling)
        for a, b in zip(outputs(plan), outputs(fresh)):
            assert torch.equal(a, b)

    near, far, small, large = _cams(1.7), _cams(), _Grid(50, 1.0), _Grid(61, 5.0)
    outputs(plan)
    for cams, grid in ((far, large), (near, large), (near, small), (far, small)):
        plan.set_grid(grid)
        plan.set_cameras(cams)
        check(cams, grid, sampling)
    other = psfs.NEAREST + psfs.BILINEAR - sampling
    plan.set_params(sampling=other)
    check(far, small, other)


@pytest.mark.gpu
def test_the_matrices_of_a_loss():
    fr = S.config_frame(0, 1)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    shape = lambda c: (c.height, c.width, 3)
    ims = [torch.randint(0, 256, shape(c), dtype=torch.uint8, device="cuda", generator=g) for c in fr.cams]
    mus, vs = ([torch.rand(shape(c), device="cuda", generator=g) * 200 + 20 for c in fr.cams] for _ in range(2))
    labels = torch.zeros((fr.grid.nz, fr.grid.ny, fr.grid.nx), dtype=torch.uint8, device="cuda")
    plan = psfs.DiffPlan(fr.cams, fr.grid)
    P = torch.from_numpy(np.stack([c.P for c in fr.cams])).cuda()
    lmap = None
    for scale in (1.0, 1.0, 2.5):                          # the last: images that show a part of the grid
        Q = P.clone()
        Q[:, :2] = Q[:, :2] * scale
        psfs.occupancy_loss(Q, mus, vs, ims, labels, plan)
        plan.set_params(sampling=psfs.NEAREST)
        lmap = plan.likelihood(ims) if lmap is None else lmap
        post, occ = plan.fuse(lmap)
        fresh = psfs.Plan([c.with_P(q) for c, q in zip(fr.cams, Q.cpu().numpy())], fr.grid)
        want, want_occ = fresh.fuse(lmap)
        assert torch.equal(post, want) and torch.equal(occ, want_occ)
        plan.set_params(sampling=psfs.BILINEAR)
