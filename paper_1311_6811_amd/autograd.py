"""Occupancy loss with gradients for calibration and background refinement.

``occupancy_loss`` wraps the library's differentiable forward (bilinear
sampling of every view's log(2*SLM) map at the projected voxel centres, mean
binary cross-entropy with logits against 0/1 labels) and its hand-written
adjoint in a ``torch.autograd.Function``. Gradients flow to the background
means and variances of every view and to the 3x4 camera matrices; images and
labels get none. Projections are recomputed in the backward, not stored.
"""
from __future__ import annotations

from typing import Optional, Sequence

import numpy as np
import torch

from . import _lib as L
from .api import LOG_U_DEFAULT, Plan, make_camera

_CAMERA = np.dtype([("width", np.int32), ("height", np.int32), ("P", np.float32, (3, 4))])   # psfs_camera


class _View:
    def __init__(self, width, height, P):
        self.width, self.height, self.P = width, height, P


class OccupancyLoss(torch.autograd.Function):
    @staticmethod
    def forward(ctx, P, plan, images, labels, sub, *bg):
        n = len(images)
        bg = [t.detach() for t in bg]
        means, vars_ = bg[:n], bg[n:]
        if plan.takes(P):
            # the matrices are read while the likelihood maps are computed
            Pd = P if P.dtype == torch.float32 and P.is_contiguous() else P.detach().to(torch.float32).contiguous()
            cams, logits, loss, ws = plan._diff_forward_at(Pd, means, vars_, images, labels, sub)
            Ph = np.frombuffer(cams, dtype=_CAMERA, count=n)["P"]
            views = [_View(c.width, c.height, Ph[k]) for k, c in enumerate(plan.sizes)]
            plan._took_views(views, means, vars_)
        else:
            Ph = P.detach().to("cpu", torch.float32).numpy().reshape(n, 3, 4).copy()
            views = [_View(c.width, c.height, Ph[k]) for k, c in enumerate(plan.sizes)]
            cams = (L.psfs_camera * max(n, 1))(*[make_camera(c.width, c.height, c.P) for c in views])
            plan._set_views(views, cams, means, vars_)
            logits, loss, ws = plan.diff_forward(images, labels, sub)
        # The plan is shared: another forward may re-set its cameras and
        # backgrounds before this backward runs, so keep this call's own
        # (host FP32 matrices, the background tensors) and re-set them there.
        ctx.plan, ctx.images, ctx.sub, ctx.ws = plan, images, sub, ws
        ctx.views, ctx.cams, ctx.bg = views, cams, (means, vars_)
        ctx.p_device = P.device
        ctx.save_for_backward(labels, logits)
        return loss

    @staticmethod
    def backward(ctx, grad_loss):
        labels, logits = ctx.saved_tensors
        ctx.plan._set_views(ctx.views, ctx.cams, *ctx.bg)
        gmeans, gvars, gP = ctx.plan.diff_backward(ctx.images, labels, logits, grad_loss, ctx.ws, ctx.sub)
        return (gP if gP.device == ctx.p_device else gP.to(ctx.p_device), None, None, None, None, *gmeans, *gvars)


class DiffPlan(Plan):
    """A plan whose cameras are re-set from a parameter tensor on each call."""

    def __init__(self, sizes: Sequence, grid, prior=0.5, log_u=LOG_U_DEFAULT):
        super().__init__(None, grid, prior=prior, log_u=log_u, sampling=L.BILINEAR)
        self.sizes = list(sizes)

    def takes(self, P: torch.Tensor) -> bool:
        """P holds a 3 x 4 matrix per view on the current GPU and the plan's
        cameras have this plan's sizes (they do after its first call): the
        forward can then read the matrices beside its own work."""
        return (P.is_cuda and P.get_device() == torch.cuda.current_device() and P.numel() == 12 * len(self.sizes)
                and self._hw == [(c.height, c.width) for c in self.sizes])


def occupancy_loss(P: torch.Tensor, means: Sequence[torch.Tensor], vars_: Sequence[torch.Tensor],
                   images: Sequence[torch.Tensor], labels: torch.Tensor, plan: DiffPlan,
                   sub: Optional[Sequence[int]] = None) -> torch.Tensor:
    """Mean BCE-with-logits occupancy loss; differentiable in P ([n][3][4]),
    means and variances (each [H][W][3], on the GPU)."""
    if P.shape != (len(images), 3, 4):
        raise ValueError(f"P must be [{len(images)}, 3, 4], got {tuple(P.shape)}")
    return OccupancyLoss.apply(P, plan, list(images), labels, None if sub is None else list(sub),
                               *means, *vars_)
