"""Bilinear sampling divides by the depth to the last bit of FP64: coordinates
k + t / c at k = 40000, whose fractions t / c of ~1e-8 px a map value of 2^28
turns into logits near 1. Every operand is exact in FP64 but for the
reciprocal of the depth and one product, which may be off by half an ulp each:
|u| 2^-52 px in all. (The hardware reciprocal with one Newton step is off by
2e-15, nine times that.)"""
import numpy as np
import pytest
import torch

import paper_1311_6811_amd as psfs
from synth import scene as S

pytestmark = pytest.mark.gpu

K, T, SCALE = 40000, 2.0 ** -27, 2.0 ** 28


class _Grid:
    nx, ny, nz, voxel = 64, 3, 64, 2.0 ** -6
    origin = np.array([0.0, 0.0, 1.0], np.float32)


def test_coordinates_to_the_last_bits():
    # depth c = Z + X / 256, u = k + t / c, v = 0
    P = np.array([[K / 256.0, 0, K, T], [0, 0, 0, 0], [1 / 256.0, 0, 1, 0]], np.float32)
    cam = S.ring_rig(1, 100.0, K + 2, 2)[0].with_P(P)
    plan = psfs.Plan([cam], _Grid, sampling=psfs.BILINEAR)
    lmap = torch.zeros(plan.lmap_floats(), device="cuda")
    plan.lmap_view(lmap, 0)[:, K + 1] = SCALE
    x, z = ((np.arange(64) + 0.5) / 64).astype(np.longdouble), (1 + (np.arange(64) + 0.5) / 64).astype(np.longdouble)
    c = z[:, None, None] + x[None, None, :] / 256 + np.zeros((1, 3, 1), np.longdouble)
    want = (1 / (1 + np.exp(-SCALE * T / c))).astype(np.float64)
    tol = 0.25 * SCALE * (K + 1) * 2.0 ** -52 + 2e-6         # 2e-6: FP32 sample, sum and sigmoid
    fused = plan.fuse(lmap)[0]
    stepped = torch.empty_like(fused)
    plan.pipeline_step(None, None, lmap, stepped)
    for post in (fused, stepped):
        err = float(np.abs(post.cpu().numpy().astype(np.float64) - want).max())
        print(f"max error {err:.2e}, allowed {tol:.2e}", flush=True)
        assert err <= tol
