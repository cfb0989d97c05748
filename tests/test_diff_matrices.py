"""Camera tensors that do not hold 3 x 4 numbers per view, given to the autograd
function itself (occupancy_loss checks their shape first): they are refused as
host tensors are, and never read as matrices on the GPU."""
import numpy as np
import pytest
import torch

import paper_1311_6811_amd as psfs
from gpu_util import upload
from synth import scene as S


class _OnGpu:
    """What DiffPlan.takes looks at of a GPU tensor."""
    is_cuda = True

    def __init__(self, *shape):
        self.shape = shape

    def get_device(self):
        return 0

    def numel(self):
        return int(np.prod(self.shape))

    def dim(self):
        return len(self.shape)

    def __len__(self):
        return self.shape[0]


def test_only_whole_matrices_are_read_on_the_gpu(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    fr = S.config_frame(0, 0)
    plan = psfs.DiffPlan(fr.cams, fr.grid)
    plan.set_cameras(fr.cams)
    n = len(fr.cams)
    assert plan.takes(_OnGpu(n, 3, 4)) and plan.takes(_OnGpu(n, 12))
    for shape in ((n, 3, 3), (n, 4, 4), (n, 1), (n, 3, 5), (n - 1, 3, 4), ()):
        assert not plan.takes(_OnGpu(*shape)), shape


@pytest.mark.gpu
def test_other_shapes_are_refused():
    fr = S.config_frame(0, 1)
    ims, mus, vs = upload(fr)
    labels = torch.from_numpy(S.gt_occupancy(fr.grid, fr.body)).cuda()
    P = torch.from_numpy(np.stack([c.P for c in fr.cams])).cuda()
    plan = psfs.DiffPlan(fr.cams, fr.grid)
    args = (plan, ims, labels, None, *mus, *vs)
    good = psfs.OccupancyLoss.apply(P, *args)
    for bad in (torch.zeros(4, 4, 4, device="cuda"), torch.zeros(4, 3, 3, device="cuda")):
        for Q in (bad, bad.cpu()):
            with pytest.raises(ValueError):
                psfs.OccupancyLoss.apply(Q, *args)
    assert torch.equal(psfs.OccupancyLoss.apply(P.view(4, 12), *args), good)
