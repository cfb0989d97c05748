"""Posteriors and occupancies of the two- and four-frame steps, stored in
16-byte pieces of rows of any length and occupancies at any address: bit-identical to the frames
alone, every voxel written and nothing beside the arrays."""
import pytest
import torch

import paper_1311_6811_amd as psfs
from tests.test_bilinear_block import _Grid, _rig

pytestmark = pytest.mark.gpu
PAD = 64


def _guarded(grid, dtype, shift, fill):
    """A volume that starts `shift` elements past an aligned address, with guards."""
    n = grid.nx * grid.ny * grid.nz
    buf = torch.full((n + 2 * PAD,), fill, dtype=dtype, device="cuda")
    return buf, buf[PAD + shift:PAD + shift + n].view(grid.nz, grid.ny, grid.nx)


@pytest.mark.parametrize("frames", [2, 4])
@pytest.mark.parametrize("nx,ny,nz,shift", [
    (64, 16, 8, 0), (48, 18, 9, 0),                  # aligned rows; whole and partial waves
    (64, 16, 8, 4), (32, 8, 4, 12),                  # occupancies at other addresses
    (33, 9, 5, 0), (35, 10, 7, 4), (34, 17, 4, 8),   # one voxel and more past a wave's 32
    (31, 16, 8, 0), (63, 2, 4, 4), (65, 3, 4, 0), (101, 7, 13, 12),
])
def test_row_pieces(frames, nx, ny, nz, shift):
    grid = _Grid(nx, ny, nz, 2.0)
    plan = psfs.Plan(_rig("ring", 5, 160, 120), grid)
    g = torch.Generator(device="cuda")
    g.manual_seed(nx * 10 + shift)
    maps = -6.0 * torch.rand(frames * max(plan.lmap_floats(), 4), device="cuda", generator=g) + 0.6
    posts = [_guarded(grid, torch.float32, shift, -1.0) for _ in range(frames)]
    occs = [_guarded(grid, torch.uint8, (shift + 5 * f + 1) % 16 if shift else 0, 7) for f in range(frames)]
    if frames == 2:
        plan.pipeline_step_pair(None, None, None, maps, posts[0][1], occs[0][1], posts[1][1], occs[1][1])
    else:
        plan.pipeline_step_quad(None, None, maps, [p for _, p in posts], [o for _, o in occs])
    for f in range(frames):
        ref, ref_occ = plan.fuse(maps.view(-1, frames)[:, f].contiguous())
        assert torch.equal(posts[f][1], ref) and torch.equal(occs[f][1], ref_occ), f
        assert int((posts[f][0] == -1.0).sum()) == 2 * PAD, f
        assert int((occs[f][0] == 7).sum()) == 2 * PAD, f
