"""Smoothing in 16-byte pieces against the scalar kernel (which a posterior at
an odd address takes), and the foreground histogram of 16-pixel pieces against
a plain count, where their pieces, lane groups and tails can go wrong."""
import numpy as np
import pytest
import torch

import paper_1311_6811_amd as psfs
from synth import scene as S

pytestmark = pytest.mark.gpu


def _plan(nx, ny, nz):
    voxel = np.float32(0.01)
    return psfs.Plan([], S.Grid(nx, ny, nz, np.zeros(3, np.float32), voxel))


@pytest.mark.parametrize("nx,ny,nz", [(4, 1, 1), (4, 3, 2), (60, 5, 3), (64, 8, 4), (68, 9, 5), (124, 7, 1), (128, 2, 6),
                                      (132, 3, 3), (256, 5, 2), (260, 4, 3), (516, 3, 3)])
def test_smoothing_pieces_have_the_scalar_kernels_bits(nx, ny, nz):
    plan = _plan(nx, ny, nz)
    g = torch.Generator(device="cuda")
    g.manual_seed(nx + 1000 * ny)
    n = nx * ny * nz
    buf = torch.empty(n + 1, device="cuda")
    buf[1:] = torch.rand(n, device="cuda", generator=g) ** 2
    odd = buf[1:].view(nz, ny, nx)                   # 4 bytes past a 16-byte boundary: scalar kernel
    even = odd.clone()
    a, b = plan.surface(even, want_smoothed=True), plan.surface(odd, want_smoothed=True)
    assert torch.equal(a.smoothed, b.smoothed) and torch.equal(a.occ, b.occ)
    assert torch.equal(a.indices(), b.indices())
    # 27 in-grid values, each rounded once, summed and divided in FP32
    p = even.double().cpu()[None, None]
    box, ones = torch.ones((1, 1, 3, 3, 3), dtype=torch.float64), torch.ones_like(p)
    want = torch.nn.functional.conv3d(p, box, padding=1) / torch.nn.functional.conv3d(ones, box, padding=1)
    assert float((a.smoothed.cpu().double() - want[0, 0]).abs().max()) <= 27 * 2.0 ** -24


@pytest.mark.parametrize("w,h,off,use_map", [(1, 1, 0, False), (15, 1, 1, False), (16, 1, 3, False), (17, 5, 2, True),
                                             (129, 127, 0, True), (131, 125, 7, False), (257, 256, 0, False)])
def test_foreground_counts(w, h, off, use_map):
    cams = S.ring_rig(2, 100.0, w, h)
    plan = psfs.Plan(cams)
    rng = np.random.default_rng(w * 7 + h)
    imgs = [rng.integers(0, 256, (h, w, 3), dtype=np.uint8) for _ in cams]
    marks = [rng.random((h, w)) < 0.4 for _ in cams]
    if w * h < 20:
        marks[1][:] = False                          # a view without foreground
    ims = [torch.from_numpy(i).cuda() for i in imgs]
    if use_map:
        lmap = torch.full((plan.lmap_floats(),), 1.0, device="cuda")      # padding that must not count
        for k, m in enumerate(marks):
            plan.lmap_view(lmap, k)[:] = torch.from_numpy(np.where(m, 0.5, 0.0).astype(np.float32)).cuda()
        out = plan.foreground_model(ims, lmap=lmap)
    else:
        masks = []
        for m in marks:
            buf = torch.zeros(w * h + 16, dtype=torch.uint8, device="cuda")
            buf[off:off + w * h] = torch.from_numpy(m.astype(np.uint8).ravel() * 200).cuda()
            buf[off + w * h:] = 1
            masks.append(buf[off:off + w * h].view(h, w))
        out = plan.foreground_model(ims, masks=masks)
    b = np.concatenate([i[m] for i, m in zip(imgs, marks)]).astype(np.int64) >> 4
    c = np.bincount(b[:, 0] * 256 + b[:, 1] * 16 + b[:, 2], minlength=4096).astype(np.float64)
    want = np.log((c + 1.0) / ((c.sum() + 4096.0) * 4096.0))
    # the FP64 logarithm rounded to FP32
    assert np.max(np.abs(out.cpu().numpy() / want - 1.0)) <= 2.0 ** -24 + 1e-15
