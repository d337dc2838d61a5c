"""torch.autograd wrapper of the likelihood: forward smc_loglik, or where a
gradient may follow smc_loglik_ckpt, whose checkpoints are saved for the
backward (smc_loglik_backward_ckpt, the hand-written adjoint), so that the
recursion runs forward once.  Marshalling only."""
from __future__ import annotations

import torch

from . import _lib


class SmcLoglik(torch.autograd.Function):
    """loglik[p] = log p(y_{1:t} | theta[:, p]) for theta of shape [d, P]
    (FP64, on the model's device)."""

    @staticmethod
    def forward(ctx, theta, model, t):
        theta = theta.contiguous()
        ctx.model, ctx.t = model, t
        if not ctx.needs_input_grad[0]:
            return _lib.smc_loglik(model, theta, t)
        ll, ckpt = _lib.smc_loglik_ckpt(model, theta, t)
        ctx.save_for_backward(theta, ckpt)
        return ll

    @staticmethod
    def backward(ctx, grad_out):
        theta, ckpt = ctx.saved_tensors
        dtheta = _lib.smc_loglik_backward_ckpt(ctx.model, theta, ctx.t,
                                               grad_out.contiguous().to(torch.float64), ckpt)
        return dtheta, None, None


def loglik(theta, model, t):
    # without a graph no gradient can follow: no checkpoints to leave
    return SmcLoglik.apply(theta if torch.is_grad_enabled() else theta.detach(), model, t)
