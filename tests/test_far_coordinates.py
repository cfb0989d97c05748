"""Pixel coordinates past the range of an int, infinite and not a number: no view
sees such a voxel, on any path, and the colour step agrees. (A coordinate that
wrapped instead of saturating would land in the image for some of the voxels.)"""
import numpy as np
import pytest
import torch

import paper_1311_6811_amd as psfs
from synth import scene as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("row,beyond", [
    ([3e7, 2e7, 1e7, 4e12], True), ([-3e7, -2e7, -1e7, -4e12], True),      # up to 1e12 pixels
    ([1e38, 1e38, 1e38, 3e38], True),                                      # infinite
    ([3e38, -3e38, 0.0, 0.0], True),                                       # infinities that cancel: not a number
    ([30.0, 20.0, 10.0, 2000.0], False)])
def test_no_pixel(row, beyond):
    W, H = 60000, 40
    P = np.array([row, [0, 0, 0, 20.0], [0, 0, 0.001, 1.0]], np.float32)
    grid = S.Grid(96, 80, 64, np.array([500.0, 500.0, 1.0], np.float32), np.float32(1.0))
    plan = psfs.Plan([S.ring_rig(1, 100.0, W, H)[0].with_P(P)], grid)
    lmap = torch.full((plan.lmap_floats(),), -2.0, device="cuda")
    outs = []
    for tile in range(-1, len(psfs.tiles())):
        plan.set_tile(tile)
        post, _ = plan.fuse(lmap)
        step = torch.empty_like(post)
        plan.pipeline_step(None, None, lmap, step)
        outs += [post, step]
    more = [torch.empty_like(post) for _ in range(6)]
    plan.pipeline_step_pair(None, None, None, lmap.repeat(2), more[0], None, more[1], None)
    plan.pipeline_step_quad(None, None, lmap.repeat(4), more[2:], None)
    seen = int((outs[0] != 0.5).sum())
    assert (seen == 0) if beyond else (seen > 1000)
    for o in outs + more:
        assert torch.equal(o, outs[0])
    voxels = torch.arange(0, 96 * 80 * 64, 7, dtype=torch.int32, device="cuda")
    img = torch.full((H, W, 3), 9, dtype=torch.uint8, device="cuda")
    colour, views = plan.colour([img], voxels)
    assert not beyond or (int(views.sum()) == 0 and float(colour.abs().max()) == 0.0)
