"""torch.autograd wrapper with first and second derivatives.

Forward: Y = sph(xyz), values only.  The backward forms the derivatives again
from the points, in registers, and contracts them with the upstream gradient
(sph_vector_jacobian): storing dY in the forward and reading it back would
move seven times the bytes.  That backward is itself a differentiable
function of (grad_Y, xyz) whose derivatives come from sph_double_backward, so
forces trained through an energy (double backward) work.  All arithmetic runs
in the HIP kernels.
"""
from __future__ import annotations

import torch

from . import _native


class _SphBackward(torch.autograd.Function):
    @staticmethod
    def forward(ctx, grad_Y, xyz, l_max, normalize):
        ctx.save_for_backward(grad_Y, xyz)
        ctx.l_max = l_max
        ctx.normalize = normalize
        # (contiguous: as saved, unless saved-tensor hooks gave another layout back)
        return _native.sph_vector_jacobian(xyz.contiguous(), grad_Y.contiguous(), l_max, normalize)

    @staticmethod
    def backward(ctx, v):
        grad_Y, xyz = ctx.saved_tensors
        want_gg = ctx.needs_input_grad[0]
        want_x = ctx.needs_input_grad[1]
        if not (want_gg or want_x):
            return None, None, None, None
        ggY, g2 = _native.sph_double_backward(xyz.contiguous(), grad_Y.contiguous(), v.contiguous(), ctx.l_max,
                                              ctx.normalize, want_grad_grad_Y=want_gg, want_grad_xyz=want_x)
        return ggY, g2, None, None


class _Sph(torch.autograd.Function):
    @staticmethod
    def forward(ctx, xyz, l_max, normalize):
        ctx.l_max = l_max
        ctx.normalize = normalize
        ctx.save_for_backward(xyz)
        return _native.sph_compute(xyz, l_max, normalize)

    @staticmethod
    def backward(ctx, grad_Y):
        (xyz,) = ctx.saved_tensors
        return _SphBackward.apply(grad_Y, xyz, ctx.l_max, ctx.normalize), None, None


def spherical_harmonics(xyz: torch.Tensor, l_max: int, normalize: bool = True) -> torch.Tensor:
    """Y[n,(l_max+1)^2] for points xyz[n,3]; differentiable twice w.r.t. xyz.

    ``normalize=False`` gives the scaled (solid) harmonics r^l Y_l^m.
    """
    return _Sph.apply(xyz.contiguous(), int(l_max), bool(normalize))


def spherical_harmonics_with_gradients(xyz: torch.Tensor, l_max: int, normalize: bool = True):
    """(Y, dY) without autograd: dY[n,3,K] = dY/dxyz from the same pass."""
    with torch.no_grad():
        return _native.sph_compute_with_gradients(xyz.contiguous(), l_max, normalize)


class _SphE3nn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, xyz, l_max, normalize, normalization):
        ctx.args = l_max, normalize, normalization
        xp = _native.sph_e3nn_coordinates(xyz)  # a copy: the backward does not depend on the caller's tensor
        ctx.save_for_backward(xp)
        return _native.sph_e3nn_compute(xp, l_max, normalize, normalization)

    @staticmethod
    def backward(ctx, grad_Y):
        (xp,) = ctx.saved_tensors
        return _native.sph_e3nn_vector_jacobian(xp.contiguous(), grad_Y.contiguous(), *ctx.args), None, None, None


def e3nn_spherical_harmonics(xyz: torch.Tensor, l_max: int, normalize: bool = True,
                             normalization: str = "integral") -> torch.Tensor:
    """Y[n,(l_max+1)^2] in e3nn's convention (Sec. III.B): degrees 0..l_max,
    y as the polar axis, ``normalization`` "integral", "component" or
    "norm"; differentiable once w.r.t. xyz.  The points are permuted once; the
    forward and the backward apply the factors as they form the values and
    derivatives (include/sph.h: sph_e3nn_coordinates, sph_e3nn_compute,
    sph_e3nn_vector_jacobian)."""
    if normalization not in _native.E3NN_NORMALIZATIONS:
        raise ValueError(f"normalization must be one of {sorted(_native.E3NN_NORMALIZATIONS)}")
    return _SphE3nn.apply(xyz.contiguous(), int(l_max), bool(normalize), normalization)


def e3nn_spherical_harmonics_with_gradients(xyz: torch.Tensor, l_max: int, normalize: bool = True,
                                            normalization: str = "integral"):
    """(Y, dY) in e3nn's convention without autograd; dY[n,3,K] along x, y, z."""
    with torch.no_grad():
        xp = _native.sph_e3nn_coordinates(xyz.contiguous())
        Y, dY = _native.sph_compute_with_gradients(xp, l_max, normalize)
        return _native.sph_e3nn_convert(Y, dY, l_max, normalization)


class SphericalHarmonics(torch.nn.Module):
    """Module form: ``SphericalHarmonics(l_max, normalize)(xyz) -> Y``."""

    def __init__(self, l_max: int, normalize: bool = True):
        super().__init__()
        if not 0 <= int(l_max) <= 32:
            raise ValueError("l_max must be in [0, 32]")
        self.l_max = int(l_max)
        self.normalize = bool(normalize)

    def forward(self, xyz: torch.Tensor) -> torch.Tensor:
        return spherical_harmonics(xyz, self.l_max, self.normalize)

    def compute_with_gradients(self, xyz: torch.Tensor):
        return spherical_harmonics_with_gradients(xyz, self.l_max, self.normalize)

    def extra_repr(self) -> str:
        return f"l_max={self.l_max}, normalize={self.normalize}"
