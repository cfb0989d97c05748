"""Bilinear boxes staged in 16-byte pieces or pixel by pixel: the widths around
whole pieces, with boxes at every border of the images, give the bits of the
column kernel (the fusion inside a step) and the same logits in the
differentiable forward."""
import pytest
import torch

import paper_1311_6811_amd as psfs
from tests.test_bilinear_block import _Grid, _rig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(96, 70), (97, 70), (98, 71), (99, 70), (100, 69), (5, 4), (4, 3), (3, 5)])
@pytest.mark.parametrize("kind,side", [("ring", 2.0), ("ring", 6.0), ("close", 2.0)])
def test_widths_around_whole_pieces(W, H, kind, side):
    cams = _rig(kind, 5, W, H)
    plan = psfs.Plan(cams, _Grid(40, 33, 19, side), sampling=psfs.BILINEAR)
    g = torch.Generator(device="cuda")
    g.manual_seed(W)
    images = [torch.randint(0, 256, (H, W, 3), dtype=torch.uint8, device="cuda", generator=g) for _ in cams]
    plan.set_backgrounds([255 * torch.rand(H, W, 3, device="cuda", generator=g) for _ in cams],
                         [25 + 200 * torch.rand(H, W, 3, device="cuda", generator=g) for _ in cams])
    lmap = plan.likelihood(images)
    post, occ = plan.fuse(lmap)
    ref, ref_occ = torch.empty_like(post), torch.empty_like(occ)
    plan.pipeline_step(None, None, lmap, ref, ref_occ)
    assert torch.equal(post, ref) and torch.equal(occ, ref_occ)
    logits = plan.diff_forward(images, occ)[0]
    # the posterior is the sigmoid of the same logits, evaluated by the fast exponential
    assert torch.allclose(torch.sigmoid(logits.double()), post.double(), rtol=0, atol=2e-6)
