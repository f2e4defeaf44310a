"""torch.autograd.Function over the hsbuild forward and its hand-written adjoint.

HSBuildFunction.apply(tau, T, builder, k_frac, g) returns the full Hermitian
H and S (mirrored from the upper triangles the library writes); backward
passes the Hermitian parts of the incoming gradients to hsbuild_backward,
which recomputes the coefficients instead of keeping them.  The Hermitian
part is exact for tau and for every Hermitian direction of T.
"""
from __future__ import annotations

import torch

from .hsbuild import HSBuilder


class HSBuildFunction(torch.autograd.Function):
    @staticmethod
    def forward(ctx, tau: torch.Tensor, T: torch.Tensor, builder: HSBuilder, k_frac, g: torch.Tensor):
        H, S = builder.forward(k_frac, g, tau.detach(), T.detach())
        ctx.builder = builder
        ctx.k_frac = tuple(float(x) for x in k_frac)
        ctx.save_for_backward(tau.detach(), T.detach(), g)
        return builder.mirror(H, S)

    @staticmethod
    def backward(ctx, gH, gS):
        tau, T, g = ctx.saved_tensors
        gH, gS = ctx.builder.hermitian_part(int(g.shape[0]), gH, gS)
        gT, gtau = ctx.builder.backward(ctx.k_frac, g, tau, T, gH, gS)
        return gtau, gT, None, None, None


def hs_build(tau: torch.Tensor, T: torch.Tensor, builder: HSBuilder, k_frac, g: torch.Tensor):
    """Differentiable (H, S) as full Hermitian matrices."""
    return HSBuildFunction.apply(tau, T, builder, k_frac, g)
