"""Differentiable bit-reversed permutation for PyTorch.

``BitRev.apply(x)`` permutes the last dimension of ``x`` (length 2^k) row by
row with the library's ``bitrev_rows`` kernel.  The permutation matrix P
satisfies P^T = P because rev_k(rev_k(i)) = i (arXiv:1708.01873,
Introduction), so the backward applies the same kernel to the incoming
gradient: dL/dx = P^T g = P g.  Nothing is saved for backward.
"""
from __future__ import annotations

import torch

from . import _check, _current_stream, _load, _tensor_args


def _log2_last(x: torch.Tensor) -> int:
    if x.dim() == 0:
        raise ValueError("BitRev needs at least one dimension")
    n = x.shape[-1]
    k = int(n).bit_length() - 1
    if n <= 0 or (1 << k) != n:
        raise ValueError("last dimension %d is not a power of two" % n)
    return k


def _permute(x: torch.Tensor) -> torch.Tensor:
    k = _log2_last(x)
    # the kernel reads memory: a conjugate or negative that torch keeps as a
    # bit of the tensor (contiguous() keeps it too) is written out first
    x = x.resolve_conj().resolve_neg().contiguous()
    y = torch.empty_like(x)
    if x.numel():
        src, size = _tensor_args(x, "src")
        _check(_load().bitrev_rows(src, y.data_ptr(), k, x.numel() >> k, size, _current_stream()),
               "bitrev_rows")
    return y


def _unknown() -> bool:
    return True


def _recorded() -> bool:
    """Whether grad mode, a functorch transform, a forward-mode level or a
    trace sees what is computed now.  Torch has no public names for the last
    three: a build without one of these counts as recording."""
    return (torch.is_grad_enabled()
            or getattr(torch._C, "_are_functorch_transforms_active", _unknown)()
            or getattr(torch.autograd.forward_ad, "_current_level", 0) >= 0
            or getattr(torch._C, "_get_tracing_state", _unknown)() is not None)


class BitRev(torch.autograd.Function):
    """y[..., rev(j)] = x[..., j]; backward: the same permutation of grad."""

    @staticmethod
    def forward(ctx, x: torch.Tensor) -> torch.Tensor:
        return _permute(x)

    @staticmethod
    def backward(ctx, grad: torch.Tensor) -> torch.Tensor:
        # The adjoint is the permutation itself; applying it through BitRev
        # keeps higher-order gradients available.  Where nothing can record
        # it, the kernel is called directly: the nested apply on the engine's
        # thread cost 40 of the 111 us of a forward and backward.
        return BitRev.apply(grad) if _recorded() else _permute(grad)


def bitrev(x: torch.Tensor) -> torch.Tensor:
    """Differentiable bit-reversed permutation of the last dimension."""
    return BitRev.apply(x)
