"""torch.autograd binding of the smooth statistic.

The forward pass calls the library's hand-written gradient kernel (stt_grad) when theta asks for a
gradient and autograd records, its forward kernel (stt_smooth) otherwise; the backward pass scales the gradient by the
incoming one. Nothing is differentiated by torch itself. stt_grad gives the same statistic in the
same kernel time as stt_smooth (16 us for 1024 templates on 1000 x 1000), so a launch of its own in
the backward pass, and the host work around it, would be paid for nothing.
"""
from __future__ import annotations

import torch


class SmoothSNR(torch.autograd.Function):
    """z~(theta) per template: theta [n][6] float32 (tau0, tau2, phi0, phi1, phi2, dtau_ms), K [n] int32."""

    @staticmethod
    def forward(fctx, theta, K, ctx, m, record=True):
        theta_c = theta.detach().contiguous()
        # needs_input_grad is set for a leaf under no_grad too (64 templates: 12.8 us with the gradient, 11.0 without)
        if not (record and fctx.needs_input_grad[0]):
            return ctx.smooth(m, theta_c, K)
        z, g = ctx.grad(m, theta_c, K)
        # theta and K are saved for autograd's check that neither was modified in place
        fctx.save_for_backward(theta_c, K, g)
        return z

    @staticmethod
    def backward(fctx, gz):
        _, _, g = fctx.saved_tensors
        return gz.to(g.dtype)[:, None] * g, None, None, None, None


def smooth_snr(ctx, m, theta: torch.Tensor, K: torch.Tensor) -> torch.Tensor:
    if torch.is_grad_enabled():
        return SmoothSNR.apply(theta, K, ctx, m)
    return SmoothSNR.apply(theta, K, ctx, m, False)
