"""One-frame steps on every tile and on the tile that the plan picks: the
likelihood rounds of workgroups of two and of four waves, at pixel counts around
theirs, and the fusion beside them, bit-identical to the separate calls."""
import numpy as np
import pytest
import torch

import paper_1311_6811_amd as psfs
from tests.test_bilinear_block import _Grid, _rig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,n,W,H", [
    (9, 17, 5, 1, 16, 16), (8, 16, 4, 3, 32, 16),    # one wave, one workgroup of two
    (40, 33, 20, 2, 33, 16), (33, 15, 9, 5, 64, 16), # ragged; one workgroup of four waves
    (64, 64, 64, 4, 41, 25), (65, 64, 64, 4, 160, 119),   # 512 tiles of 8 x 16 columns and more
    (24, 40, 12, 16, 61, 67),
])
@pytest.mark.parametrize("sampling", [psfs.NEAREST, psfs.BILINEAR])
def test_step_on_every_tile(nx, ny, nz, n, W, H, sampling):
    rng = np.random.default_rng(nx + W)
    cams = _rig("ring", n, W, H)
    plan = psfs.Plan(cams, _Grid(nx, ny, nz, 2.0), sampling=sampling)
    plan.set_backgrounds([torch.from_numpy((255 * rng.random((H, W, 3))).astype(np.float32)).cuda() for _ in cams],
                         [torch.from_numpy((25 + 200 * rng.random((H, W, 3))).astype(np.float32)).cuda() for _ in cams])
    a, b = ([torch.from_numpy(rng.integers(0, 256, (H, W, 3), dtype=np.uint8)).cuda() for _ in cams] for _ in range(2))
    cur, ref_next = plan.likelihood(a), plan.likelihood(b)
    plan.set_tile(0)
    ref, ref_occ = torch.empty((nz, ny, nx), device="cuda"), torch.empty((nz, ny, nx), dtype=torch.uint8, device="cuda")
    plan.pipeline_step(None, None, cur, ref, ref_occ)
    for tile in range(-1, len(psfs.tiles())):
        plan.set_tile(tile)
        post, occ, nxt = torch.full_like(ref, -1.0), torch.full_like(ref_occ, 7), plan.new_lmap()
        plan.pipeline_step(b, nxt, cur, post, occ)
        assert torch.equal(post, ref) and torch.equal(occ, ref_occ), tile
        for v in range(n):
            assert torch.equal(plan.lmap_view(nxt, v), plan.lmap_view(ref_next, v)), (tile, v)
        if sampling == psfs.NEAREST:
            post, occ = plan.fuse(cur)
            assert torch.equal(post, ref) and torch.equal(occ, ref_occ), tile
