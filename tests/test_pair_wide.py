"""Two-frame fusion from a view of 2^29 pixels or more, whose pair map needs more
than 32 bits of byte offsets: the bits of each frame alone."""
import numpy as np
import pytest
import torch

import paper_1311_6811_amd as psfs
from synth import scene as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side", [1.5, 6.0])              # inside the image, and past its borders
def test_pair_maps_of_many_pixels(side):
    W, H = 32768, 16400
    h = np.float32(side / 36)
    grid = S.Grid(36, 33, 34, np.array([-18 * h, -16.5 * h, -17 * h], np.float32), h)
    plan = psfs.Plan(S.ring_rig(1, 0.9 * H, W, H), grid)
    n = plan.lmap_floats()
    pair = torch.empty((n, 2), device="cuda").uniform_(-6.0, 0.6)
    post = [torch.full((34, 33, 36), -1.0, device="cuda") for _ in range(2)]
    occ = [torch.full((34, 33, 36), 7, dtype=torch.uint8, device="cuda") for _ in range(2)]
    plan.pipeline_step_pair(None, None, None, pair.view(-1), post[0], occ[0], post[1], occ[1])
    for f in range(2):
        p, o = plan.fuse(pair[:, f].contiguous())
        assert torch.equal(p, post[f]) and torch.equal(o, occ[f])
        assert (int((p == 0.5).sum()) > 0) == (side > 2)
