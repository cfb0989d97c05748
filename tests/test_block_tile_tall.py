"""The block tile on boxes far down a tall image and as wide as their rows are
many pixels: row times width passes 2^24, where FP32 no longer holds every
integer. The same bits as the column tile, which indexes in integers."""
import numpy as np
import pytest
import torch

import paper_1311_6811_amd as psfs
from synth import scene as S

pytestmark = pytest.mark.gpu


class _Grid:
    nx, ny, nz, voxel = 32, 32, 32, 1.0
    origin = np.array([-16.0, -16.0, 100.0], np.float32)


@pytest.mark.parametrize("W,H,v0", [(400, 65000, 64980.0), (400, 65000, 20.0), (403, 40000, 39990.0)])
def test_edge_boxes_past_two_to_the_24(W, H, v0):
    # ten times wider than high pixels: a block of 16 voxels covers ~300 x ~10 of them, and the grid the
    # image's right and bottom (or top) borders
    P = np.array([[1900.0, 0, 350.0, 0], [0, 30.0, v0, 0], [0, 0, 1.0, 0]], np.float32)
    cam = S.ring_rig(1, 100.0, W, H)[0].with_P(P)
    plan = psfs.Plan([cam], _Grid)
    g = torch.Generator(device="cuda")
    g.manual_seed(W)
    lmap = -6.0 * torch.rand(plan.lmap_floats(), device="cuda", generator=g) + 0.6
    plan.set_tile(0)
    ref, ref_occ = plan.fuse(lmap)
    assert int((ref != 0.5).sum()) > 1000                # some voxels are seen, some are not
    assert int((ref == 0.5).sum()) > 1000
    plan.set_tile(6)
    post, occ = plan.fuse(lmap)
    assert torch.equal(post, ref) and torch.equal(occ, ref_occ)
    post.fill_(-1.0)
    plan.pipeline_step(None, None, lmap, post, occ)
    assert torch.equal(post, ref) and torch.equal(occ, ref_occ)
