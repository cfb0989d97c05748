"""Bilinear fusion from pixel boxes staged in LDS against the column kernels
(the fusion part of the pipelined step, which gathers every tap): the same
bits on every block depth, on ragged grids, with boxes larger than the LDS
arena, and with cameras inside and past the grid."""
import numpy as np
import pytest
import torch

import paper_1311_6811_amd as psfs
from synth import scene as S

pytestmark = pytest.mark.gpu


class _Grid:
    def __init__(self, nx, ny, nz, side):
        self.nx, self.ny, self.nz, self.voxel = nx, ny, nz, side / max(nx, ny, nz)
        self.origin = np.array([-0.5 * self.voxel * d for d in (nx, ny, nz)], np.float32)


def _rig(kind, n, W, H):
    f = 0.9375 * W
    if kind == "ring":
        return S.ring_rig(n, f, W, H)
    radius = {"inside": 0.3, "close": 1.3, "far": 40.0}[kind]
    cams = S.ring_rig(n, f, W, H, radius)
    if kind == "close":                              # looks past the grid: most boxes miss the image
        cams = [c.with_P(np.array([[1, 0, 0.7 * W], [0, 1, 0], [0, 0, 1]]) @ c.P) for c in cams]
    return cams


@pytest.mark.parametrize("nx,ny,nz,n,kind,W,H", [
    (1, 1, 1, 1, "ring", 320, 240),                  # one voxel
    (17, 16, 9, 16, "ring", 320, 240),               # 2 deep, all views
    (61, 53, 47, 5, "ring", 321, 243),               # 2 deep, ragged
    (100, 90, 64, 3, "inside", 320, 240),            # 4 deep, voxels behind the cameras
    (128, 128, 66, 4, "close", 320, 240),            # 8 deep, views that leave the image
    (70, 64, 60, 6, "ring", 1283, 721),              # boxes that exceed the arena
    (128, 120, 130, 12, "far", 643, 477),            # all views in one group
    (64, 64, 64, 0, "ring", 320, 240),               # no views
])
def test_block_kernel_has_the_bits_of_the_column_kernels(nx, ny, nz, n, kind, W, H):
    cams = _rig(kind, n, W, H) if n else []
    plan = psfs.Plan(cams, _Grid(nx, ny, nz, 2.0), sampling=psfs.BILINEAR)
    g = torch.Generator(device="cuda")
    g.manual_seed(nx * 1000 + n)
    lmap = -6.0 * torch.rand(max(plan.lmap_floats(), 4), device="cuda", generator=g) + 0.6
    post, occ = plan.fuse(lmap)
    ref, ref_occ = torch.empty_like(post), torch.empty_like(occ)
    plan.pipeline_step(None, None, lmap, ref, ref_occ)
    torch.cuda.synchronize()
    assert torch.equal(post, ref) and torch.equal(occ, ref_occ)
    if n:
        assert float(post.max() - post.min()) > 0 or nx * ny * nz == 1
