"""The block tile (pixel boxes in LDS, in 16-byte pieces or pixel by pixel)
against the column tile, which gathers every pixel: the same bits at ragged
grids, at widths that are no whole pieces, at the images' borders, with boxes
larger than the arena and with cameras inside and past the grid; and the tile
that a plan and a batch pick by themselves."""
import numpy as np
import pytest
import torch

import paper_1311_6811_amd as psfs
from tests.test_bilinear_block import _Grid, _rig

pytestmark = pytest.mark.gpu
BLOCK = 6


def _maps(plan, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return -6.0 * torch.rand(max(plan.lmap_floats(), 4), device="cuda", generator=g) + 0.6


@pytest.mark.parametrize("nx,ny,nz,side,n,kind,W,H", [
    (1, 1, 1, 2.0, 1, "ring", 320, 240),             # one voxel
    (17, 16, 9, 2.0, 16, "ring", 321, 240),          # ragged, all views, odd width
    (33, 31, 40, 8.0, 7, "ring", 322, 243),          # grid larger than the images: boxes at every border
    (33, 31, 40, 8.0, 7, "ring", 323, 243),
    (33, 31, 40, 8.0, 7, "ring", 324, 243),
    (48, 48, 24, 2.0, 5, "inside", 321, 240),        # voxels behind the cameras
    (64, 40, 24, 2.0, 6, "close", 643, 477),         # views that leave the image
    (40, 48, 32, 2.0, 4, "ring", 1283, 721),         # boxes that exceed the arena
    (96, 80, 72, 2.0, 12, "far", 643, 477),          # all views in one group
    (32, 32, 32, 2.0, 0, "ring", 320, 240),          # no views
])
def test_block_tile_has_the_column_tiles_bits(nx, ny, nz, side, n, kind, W, H):
    cams = _rig(kind, n, W, H) if n else []
    plan = psfs.Plan(cams, _Grid(nx, ny, nz, side))
    lmap = _maps(plan, nx * 100 + W)
    plan.set_tile(0)
    ref, ref_occ = plan.fuse(lmap)
    for tile in (BLOCK, 1, 3, 4, -1):
        plan.set_tile(tile)
        post, occ = plan.fuse(lmap)
        assert torch.equal(post, ref) and torch.equal(occ, ref_occ), tile
        post.fill_(-1.0)
        plan.pipeline_step(None, None, lmap, post, occ)
        assert torch.equal(post, ref) and torch.equal(occ, ref_occ), tile


@pytest.mark.parametrize("N,n,W,H", [(160, 12, 640, 480), (200, 8, 427, 320), (176, 6, 1283, 721), (128, 8, 640, 480)])
def test_automatic_tile(N, n, W, H):
    cams = _rig("ring", n, W, H)
    plan = psfs.Plan(cams, _Grid(N, N, N, 2.0))
    lmap = _maps(plan, N + n)
    post, occ = plan.fuse(lmap)
    plan.set_tile(0)
    ref, ref_occ = plan.fuse(lmap)
    assert torch.equal(post, ref) and torch.equal(occ, ref_occ)


def _frames(seed, turn):
    rng = np.random.default_rng(seed)
    out = []
    for N, n, W, H in ((160, 12, 320, 240), (40, 4, 161, 119), (176, 6, 643, 477)):
        cams = _rig("ring", n, W, H)
        cams = cams[turn:] + cams[:turn]
        ims = [torch.from_numpy(rng.integers(0, 256, (H, W, 3), dtype=np.uint8)).cuda() for _ in cams]
        mus = [torch.from_numpy((255 * rng.random((H, W, 3))).astype(np.float32)).cuda() for _ in cams]
        vs = [torch.from_numpy((25 + 200 * rng.random((H, W, 3))).astype(np.float32)).cuda() for _ in cams]
        out.append(psfs.BatchFrame(cams, _Grid(N, N, N, 2.0), ims, mus, vs))
    return out


def test_batch_with_block_frames_and_an_update():
    stream = torch.cuda.Stream()
    batch = psfs.Batch(_frames(1, 0))
    for frames in (batch.frames, _frames(2, 3)):
        if frames is not batch.frames:
            batch.update(frames)
        stream.wait_stream(torch.cuda.current_stream())
        for _ in range(2):
            for f in frames:
                f.posterior.fill_(-1.0)
            stream.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(stream):
                batch.run()
            stream.synchronize()
            for f in frames:
                plan = psfs.Plan(f.cams, f.grid)
                plan.set_backgrounds(f.means, f.vars)
                plan.set_tile(0)
                post, occ = plan.reconstruct(f.images)
                assert torch.equal(post, f.posterior) and torch.equal(occ, f.occ)


@pytest.mark.parametrize("nz", [1, 3, 4, 5, 8, 12, 15, 16, 17, 31, 33])
def test_depths_that_do_not_fill_a_stack(nz):
    plan = psfs.Plan(_rig("ring", 6, 332, 250), _Grid(33, 18, nz, 2.0))
    lmap = _maps(plan, nz)
    plan.set_tile(0)
    ref, ref_occ = plan.fuse(lmap)
    plan.set_tile(BLOCK)
    post, occ = torch.full_like(ref, -1.0), torch.full_like(ref_occ, 7)
    plan.pipeline_step(None, None, lmap, post, occ)
    assert torch.equal(post, ref) and torch.equal(occ, ref_occ)
    post, occ = plan.fuse(lmap)
    assert torch.equal(post, ref) and torch.equal(occ, ref_occ)
