"""Bilinear fusion on the tile of staged pixel boxes against the column tiles,
each set by name, so that every shape runs both: all three block depths, all
views, boxes larger than the LDS arena, cameras inside and past the grid."""
import pytest
import torch

import paper_1311_6811_amd as psfs
from tests.test_bilinear_block import _Grid, _rig

pytestmark = pytest.mark.gpu
BLOCK = 6


@pytest.mark.parametrize("nx,ny,nz,n,kind,W,H", [
    (1, 1, 1, 1, "ring", 320, 240),                  # one voxel
    (17, 16, 9, 16, "ring", 320, 240),               # 2 deep, all views
    (61, 53, 47, 5, "ring", 321, 243),               # 2 deep, ragged
    (300, 290, 2, 4, "ring", 320, 240),              # 2 deep, flat
    (301, 290, 3, 4, "ring", 320, 240),              # 4 deep, flat
    (96, 90, 64, 4, "ring", 320, 240),               # 4 deep
    (100, 90, 64, 3, "inside", 320, 240),            # 4 deep, voxels behind the cameras
    (110, 81, 95, 16, "close", 643, 477),            # 4 deep, all views, most of them looking past the grid
    (128, 128, 66, 4, "close", 320, 240),            # 8 deep
    (70, 64, 60, 6, "ring", 1283, 721),              # boxes that exceed the arena
    (130, 128, 70, 7, "ring", 1283, 721),            # 8 deep, a view or two per group
    (40, 30, 20, 3, "ring", 3000, 2000),             # boxes that fit nowhere
    (64, 64, 64, 0, "ring", 320, 240),               # no views
])
def test_boxes_and_columns_have_the_same_bits(nx, ny, nz, n, kind, W, H):
    cams = _rig(kind, n, W, H) if n else []
    plan = psfs.Plan(cams, _Grid(nx, ny, nz, 2.0), sampling=psfs.BILINEAR)
    g = torch.Generator(device="cuda")
    g.manual_seed(nx * 1000 + n)
    lmap = -6.0 * torch.rand(max(plan.lmap_floats(), 4), device="cuda", generator=g) + 0.6
    plan.set_tile(0)
    ref, ref_occ = plan.fuse(lmap)
    assert n == 0 or float(ref.max() - ref.min()) > 0 or nx * ny * nz == 1
    for tile in (BLOCK, 1, 2, 3, 4, 5, -1):
        plan.set_tile(tile)
        post, occ = torch.full_like(ref, -1.0), torch.full_like(ref_occ, 7)
        plan.fuse(lmap, post, occ)
        assert torch.equal(post, ref) and torch.equal(occ, ref_occ), tile
