"""torch.autograd wrapper of the likelihood: forward smc_loglik, or where a
gradient may follow smc_loglik_ckpt, whose checkpoints are saved for the
backward (smc_loglik_backward_ckpt, the hand-written adjoint), so that the
recursion runs forward once.  Where the device has no memory for checkpoints
that live as long as the graph, theta alone is saved and the backward runs both
sweeps (smc_loglik_backward).  Marshalling only."""
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
        try:
            ll, ckpt = _lib.smc_loglik_ckpt(model, theta, t)
        except torch.OutOfMemoryError:
            ctx.save_for_backward(theta)
            return _lib.smc_loglik(model, theta, t)
        ctx.save_for_backward(theta, ckpt)
        return ll

    @staticmethod
    def backward(ctx, grad_out):
        theta, *ckpt = ctx.saved_tensors
        dloglik = grad_out.contiguous().to(torch.float64)
        if ckpt:
            return _lib.smc_loglik_backward_ckpt(ctx.model, theta, ctx.t, dloglik, ckpt[0]), None, None
        return _lib.smc_loglik_backward(ctx.model, theta, ctx.t, dloglik), None, None


def loglik(theta, model, t):
    """loglik[p] = log p(y_{1:t} | theta[:, p]), differentiable in theta.  When a
    gradient is wanted, the graph holds the adjoint's checkpoints until it is
    freed: smc_loglik_ckpt_bytes(model, P, t), for EGARCH with K factors about
    ceil(t / 32) * K * P values of the recursion's precision (1,000 FP64
    particles, K = 2, t = 1,237: 0.6 MB; 65,536 with t = 10,000: 328 MB).
    A program that keeps many graphs counts that for each.  If the forward pass
    cannot have it, the graph holds theta alone and the backward pass takes
    that much for its own duration."""
    # without a graph no gradient can follow: no checkpoints to leave
    return SmcLoglik.apply(theta if torch.is_grad_enabled() else theta.detach(), model, t)
