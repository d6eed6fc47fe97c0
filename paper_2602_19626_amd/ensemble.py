"""Softmax-gated ensemble head as a torch.autograd.Function over the library's kernels.

Experts: q_0 = softmax(z + b) (the adaptive-bias head of section 3.7 applied to the LLM logits)
and the n-gram orders P_1..P_K (section 3.5); gate w = softmax(theta); p = sum_j w_j q_j;
loss_r = -log p_r(t*_r).  Forward and backward are the hand-written kernels behind
nc_ensemble_forward / nc_ensemble_backward; the gradients are reduced over rows in a fixed order
(no float atomics).  The logits z and the n-gram experts are inputs, not parameters.
"""
from __future__ import annotations

import torch

from . import _dev_ptr, _stream_ptr
from ._lib import check, lib


def _forward(z, b, theta, P, target):
    """(loss, resp, lse) of every row: the losses, the responsibilities and logsumexp(z + b)."""
    rows, vocab = z.shape
    nexp = theta.shape[0]
    loss = torch.empty(rows, dtype=torch.float32, device=z.device)
    lse = torch.empty_like(loss)
    resp = torch.empty((rows, nexp), dtype=torch.float32, device=z.device)
    Pp = _dev_ptr(P, torch.float32, "P") if nexp > 1 else None
    check(lib().nc_ensemble_forward_lse(
        _dev_ptr(z, torch.float32, "z"), _dev_ptr(b, torch.float32, "b"),
        _dev_ptr(theta, torch.float32, "theta"), Pp, _dev_ptr(target, torch.int32, "target"),
        rows, vocab, nexp, _dev_ptr(loss, torch.float32, "loss"), _dev_ptr(resp, torch.float32, "resp"),
        _dev_ptr(lse, torch.float32, "lse"), _stream_ptr()))
    return loss, resp, lse


def _backward(z, b, theta, resp, lse, target, gl, lr, gb, gth):
    rows, vocab = z.shape
    opt = lambda t, name: None if t is None else _dev_ptr(t, torch.float32, name)
    check(lib().nc_ensemble_backward_lse(
        _dev_ptr(z, torch.float32, "z"), _dev_ptr(b, torch.float32, "b"),
        _dev_ptr(theta, torch.float32, "theta"), _dev_ptr(resp, torch.float32, "resp"),
        _dev_ptr(lse, torch.float32, "lse"), _dev_ptr(target, torch.int32, "target"),
        opt(gl, "grad_loss"), rows, vocab, theta.shape[0], float(lr), opt(gb, "grad_b"),
        opt(gth, "grad_theta"), _stream_ptr()))


class EnsembleHead(torch.autograd.Function):
    @staticmethod
    def forward(ctx, z, b, theta, P, target):
        loss, resp, lse = _forward(z, b, theta, P, target)
        ctx.save_for_backward(z, b, theta, resp, lse, target)
        return loss

    @staticmethod
    def backward(ctx, grad_loss):
        z, b, theta, resp, lse, target = ctx.saved_tensors
        gl = grad_loss.contiguous().to(torch.float32)
        gb = torch.empty_like(b)
        gth = torch.empty_like(theta)
        _backward(z, b, theta, resp, lse, target, gl, 0.0, gb, gth)
        return None, gb, gth, None, None


def ensemble_loss(z, b, theta, P, target):
    """Per-row -log p(t*) of the gated ensemble; differentiable in b and theta."""
    return EnsembleHead.apply(z, b, theta, P, target)


def ensemble_sgd_step(z, b, theta, P, target, lr: float = 1e-3):
    """One fused SGD step on (b, theta) for the summed loss, in place; returns the losses."""
    loss, resp, lse = _forward(z, b, theta, P, target)
    _backward(z, b, theta, resp, lse, target, None, lr, None, None)
    return loss
