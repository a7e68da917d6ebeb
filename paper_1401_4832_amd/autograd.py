"""torch.autograd.Function over (h, J) for the per-site objectives.

forward: f_r = B_eff * g_r^reg for every site r (eq. g_regdef2 times B_eff),
evaluated by the library's forward kernel only.  backward: the gradient
(eqs. g_gradh2, g_gradJ2), with the upstream gradient as a per-site multiplier
applied inside the library.  Where the residuals of the forward pass are small
(a workspace of at most KEEP_BYTES) they stay in its workspace for the
backward; larger ones (B*N*q values, 2.1 GB at N = 500, B = 50000) are not
kept: energies, softmax and residuals are then evaluated again.
"""
from __future__ import annotations

import torch

from . import api
from ._lib import lib, PATH_GATHER_FP32

# Most a graph holds per call between forward and backward.  At N = 150, B = 8000
# (a 234 MB workspace) a pass takes 740 us with the residuals kept;
# evaluating them again would add the forward's 425 us.
KEEP_BYTES = 1 << 30


class PLMObjective(torch.autograd.Function):
    @staticmethod
    def forward(ctx, h, J, msa, w, beff, lambda_h=0.01, lambda_J=0.01):
        ctx.lam = (lambda_h, lambda_J)
        B, N = msa.shape
        keep = (any(ctx.needs_input_grad[:2])
                and lib().plm_objgrad_workspace_bytes(B, N, h.shape[1], PATH_GATHER_FP32) <= KEEP_BYTES)
        if keep:
            f, ws = api.objgrad_begin(msa, w, beff, h.detach(), J.detach(), lambda_h, lambda_J)
            ctx.save_for_backward(h, J, msa, w, beff, ws)
        else:
            f, _, _ = api.objgrad(msa, w, beff, h.detach(), J.detach(), lambda_h, lambda_J, grad=False)
            ctx.save_for_backward(h, J, msa, w, beff)
        return f

    @staticmethod
    def backward(ctx, grad_f):
        h, J, msa, w, beff, *kept = ctx.saved_tensors
        scale = grad_f.detach().to(torch.float64).contiguous()
        # a saved-tensor hook may have handed the workspace back in another place
        if kept and kept[0].device == msa.device and kept[0].is_contiguous() and kept[0].data_ptr() % 256 == 0:
            gh, gJ = api.objgrad_finish(kept[0], msa, w, beff, h.detach(), J.detach(), *ctx.lam, grad_scale=scale)
        else:
            _, gh, gJ = api.objgrad(msa, w, beff, h.detach(), J.detach(), *ctx.lam, grad=True, grad_scale=scale)
        return gh, gJ, None, None, None, None, None


def plm_objective(h, J, msa, w, beff, lambda_h=0.01, lambda_J=0.01):
    """Per-site objectives f [N] (float64), differentiable in h [N, q] and J [N, N, q, q]."""
    return PLMObjective.apply(h, J, msa, w, beff, lambda_h, lambda_J)
