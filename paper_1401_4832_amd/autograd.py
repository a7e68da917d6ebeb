"""torch.autograd.Function over (h, J) for the per-site objectives.

forward: f_r = B_eff * g_r^reg for every site r (eq. g_regdef2 times B_eff),
evaluated by the library's forward kernel only.  backward: the gradient
(eqs. g_gradh2, g_gradJ2), with the upstream gradient as a per-site multiplier
applied inside the library.  The residuals of a forward pass (84 bytes per
sequence and site) stay in memory for its backward as long as all graphs that
are alive hold at most KEEP_BYTES of them per device; past that, energies,
softmax and residuals are evaluated again in the backward.
"""
from __future__ import annotations

import itertools
import weakref

import torch

from . import api
from ._lib import PATH_GATHER_FP32

# Most that the graphs alive on a device hold together between forward and
# backward, so that a sum over any number of families needs no more memory than
# this on top of one evaluation's.  At N = 150, B = 8000 (118 MB) a pass takes
# 740 us with the residuals kept; evaluating them again would add the forward's
# 425 us.
KEEP_BYTES = 1 << 30

_live: dict = {}  # token -> (device, bytes) of every evaluation kept
_refs: dict = {}  # token -> weak reference to its tensor, which takes both entries out
_tokens = itertools.count()


def _reserve(device, nbytes):
    """A token for nbytes more on the device, or None where they would exceed KEEP_BYTES."""
    token = next(_tokens)
    _live[token] = (device, nbytes)  # (entered first: two threads may both be refused, never both let in)
    if sum(n for d, n in _live.copy().values() if d == device) <= KEEP_BYTES:
        return token
    del _live[token]
    return None


class PLMObjective(torch.autograd.Function):
    @staticmethod
    def forward(ctx, h, J, msa, w, beff, lambda_h=0.01, lambda_J=0.01):
        ctx.lam = (lambda_h, lambda_J)
        B, N = msa.shape
        token = None
        if any(ctx.needs_input_grad[:2]):
            token = _reserve(msa.device, api.objgrad_half_sizes(B, N, h.shape[1], PATH_GATHER_FP32)[0])
        if token is not None:
            try:
                f, kept = api.objgrad_begin(msa, w, beff, h.detach(), J.detach(), lambda_h, lambda_J)
            except BaseException:
                _live.pop(token, None)
                raise
            # given back when the graph, or whoever holds the tensor, lets it go
            _refs[token] = weakref.ref(kept, lambda _, t=token: (_live.pop(t, None), _refs.pop(t, None)))
            ctx.save_for_backward(h, J, msa, w, beff, kept)
        else:
            f, _, _ = api.objgrad(msa, w, beff, h.detach(), J.detach(), lambda_h, lambda_J, grad=False)
            ctx.save_for_backward(h, J, msa, w, beff)
        return f

    @staticmethod
    def backward(ctx, grad_f):
        h, J, msa, w, beff, *kept = ctx.saved_tensors
        scale = grad_f.detach().to(torch.float64).contiguous()
        # a saved-tensor hook may have handed the residuals back in another place
        if kept and kept[0].device == msa.device and kept[0].is_contiguous() and kept[0].data_ptr() % 256 == 0:
            gh, gJ = api.objgrad_finish(kept[0], msa, w, beff, h.detach(), J.detach(), *ctx.lam, grad_scale=scale)
        else:
            _, gh, gJ = api.objgrad(msa, w, beff, h.detach(), J.detach(), *ctx.lam, grad=True, grad_scale=scale)
        return gh, gJ, None, None, None, None, None


def plm_objective(h, J, msa, w, beff, lambda_h=0.01, lambda_J=0.01):
    """Per-site objectives f [N] (float64), differentiable in h [N, q] and J [N, N, q, q]."""
    return PLMObjective.apply(h, J, msa, w, beff, lambda_h, lambda_J)
