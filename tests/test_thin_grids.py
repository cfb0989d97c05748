"""Grids of a few rows and very many planes (or the other way round), whose
workgroups reach the 2^32 lanes that one axis of a launch can have."""
import numpy as np
import pytest
import torch

import paper_1311_6811_amd as psfs
from synth import scene as S

pytestmark = pytest.mark.gpu


class _Grid:
    origin, voxel = np.zeros(3, np.float32), 1.0

    def __init__(self, nx, ny, nz):
        self.nx, self.ny, self.nz = nx, ny, nz


@pytest.mark.parametrize("nx", [1, 4])                      # row by row, and in 16-byte pieces
def test_surface_of_a_column_of_planes(nx):
    nz = 2 ** 25 + 3
    plan = psfs.Plan(grid=_Grid(nx, 1, nz), threshold=0.5)
    post = torch.full((nz, 1, nx), 0.25, device="cuda")
    post[5::7] = 1.0                                        # two thirds of the means hold one of these
    s = plan.surface(post, capacity=16)
    torch.cuda.synchronize()
    near = torch.zeros(nz, device="cuda")
    for d in (4, 5, 6):
        near[d::7] = 0.75
    want = 0.25 + near / 3.0
    want[0], want[-1] = (0.25 + 0.25) / 2, float((post[-1, 0, 0] + post[-2, 0, 0]) / 2)
    assert torch.equal(s.occ.view(nz, nx), (want[:, None] > 0.5).to(torch.uint8).expand(nz, nx))
    plan = psfs.Plan(grid=_Grid(nx, 1, nz), threshold=0.3)
    s = plan.surface(post, capacity=16, want_smoothed=True)
    assert torch.allclose(s.smoothed.view(nz, nx), want[:, None].expand(nz, nx), rtol=0, atol=1e-6)
    occ = want > 0.3
    assert torch.equal(s.occ.view(nz, nx), occ[:, None].to(torch.uint8).expand(nz, nx))
    assert int(s.count) == nx * int(occ.sum())              # every voxel is on the grid's border


@pytest.mark.parametrize("sampling", [psfs.NEAREST, psfs.BILINEAR])
def test_fusion_of_one_long_row_of_columns(sampling):
    ny = 2 ** 28
    P = np.array([[0, 0, 0, 20.0], [0, 2.0 ** -24, 0, 3.0], [0, 0, 0, 1.0]], np.float32)
    plan = psfs.Plan([S.ring_rig(1, 100.0, 40, 30)[0].with_P(P)], _Grid(1, ny, 1), sampling=sampling)
    lmap = torch.full((plan.lmap_floats(),), 0.5, device="cuda")
    post, occ = plan.fuse(lmap)
    auto = (post[0, ::4096, 0].clone(), int(occ.sum()))
    plan.set_tile(0)
    plan.fuse(lmap, post, occ)
    assert torch.equal(auto[0], post[0, ::4096, 0]) and auto[1] == int(occ.sum()) == ny
