"""The block tile set for a whole batch: every frame runs it, also small and
ragged ones, with boxes at the images' borders, boxes larger than the LDS arena
and cameras inside and past the grid. Each frame has the bits of the column
tiles."""
import numpy as np
import pytest
import torch

import paper_1311_6811_amd as psfs
from tests.test_bilinear_block import _Grid, _rig

pytestmark = pytest.mark.gpu

FRAMES = [
    (1, 1, 1, 2.0, 1, "ring", 320, 240),             # one voxel
    (17, 16, 9, 2.0, 16, "ring", 321, 240),          # ragged, all views, odd width
    (33, 31, 40, 8.0, 7, "ring", 322, 243),          # grid larger than the images: boxes at every border
    (33, 31, 40, 8.0, 7, "ring", 324, 243),
    (48, 48, 24, 2.0, 5, "inside", 321, 240),        # voxels behind the cameras
    (64, 40, 24, 2.0, 6, "close", 643, 477),         # views that leave the image
    (40, 48, 33, 2.0, 4, "ring", 1283, 721),         # boxes that exceed the arena
    (96, 80, 72, 2.0, 12, "far", 643, 477),          # all views in one group
]


def test_every_frame_on_the_block_tile():
    rng = np.random.default_rng(7)
    frames = []
    for nx, ny, nz, side, n, kind, W, H in FRAMES:
        cams = _rig(kind, n, W, H)
        ims = [torch.from_numpy(rng.integers(0, 256, (H, W, 3), dtype=np.uint8)).cuda() for _ in cams]
        mus = [torch.from_numpy((255 * rng.random((H, W, 3))).astype(np.float32)).cuda() for _ in cams]
        vs = [torch.from_numpy((25 + 200 * rng.random((H, W, 3))).astype(np.float32)).cuda() for _ in cams]
        frames.append(psfs.BatchFrame(cams, _Grid(nx, ny, nz, side), ims, mus, vs))
    refs = []
    for f in frames:
        plan = psfs.Plan(f.cams, f.grid)
        plan.set_backgrounds(f.means, f.vars)
        plan.set_tile(0)
        refs.append(plan.reconstruct(f.images))
    batch = psfs.Batch(frames)
    for tile in (6, -1, 6):
        batch.set_tile(tile)
        for f in frames:
            f.posterior.fill_(-1.0)
            f.occ.fill_(7)
        batch.run()
        for shape, f, (post, occ) in zip(FRAMES, frames, refs):
            assert torch.equal(post, f.posterior) and torch.equal(occ, f.occ), (tile, shape)
