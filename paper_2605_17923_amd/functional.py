"""torch.autograd wrappers over the C ABI: the three fused operators as differentiable functions.

Everything numerical runs in the HIP kernels; the functions allocate outputs with torch and
keep what the backward needs; the kernels round the float32 sums of the parameter gradients to the
parameters' dtype where they form them.
Inputs must be contiguous CUDA tensors in bfloat16 or float32; work is enqueued on torch's
current stream.  Without the built library every call raises (there is no fallback).

Ordinary calls run the autograd function of the C++ extension module (csrc/lnmod_torch.cpp).  The classes
below are the same functions in Python, for every call that one leaves alone: wrong arguments (they raise
the errors), tensor subclasses, functorch transforms, dispatch modes, tracers.

    y        = ln_modulate(x, shift, scale)                      x [B,S,D]; shift, scale [B,D] or [B,S,D]
    y        = ln_modulate(x, shift, scale, cu_seqlens=cu)       x [T,D] packed; shift, scale [nseg,D]
    h, y     = gated_ln_modulate(x, u, gate, shift, scale)       h = x + gate*u, y = LN(h)(1+scale)+shift
    qn, kn   = qk_norm(q, k, wq, wk)                             RMS norm with weight of q and of k
"""
import torch

from . import lnmod


def _contig(*ts):
    for t in ts:
        if t is not None and not t.is_contiguous():
            raise ValueError("tensors must be contiguous")


def _ln_backward(dy, x, scale, cu_seqlens, mean, rstd, eps):
    if cu_seqlens is not None:
        return lnmod._backward_varlen(dy, x, scale, cu_seqlens, mean, rstd, eps, io_grads=True)
    return lnmod._backward(dy, x, scale, mean, rstd, eps, io_grads=True)


class _LnModulate(torch.autograd.Function):
    """Sec. 3.3: forward saves x, scale and (optionally) the per-token statistics."""

    @staticmethod
    def forward(ctx, x, shift, scale, cu_seqlens, eps, save_stats):
        _contig(x, shift, scale, cu_seqlens)
        if cu_seqlens is None:
            y, mean, rstd = lnmod.forward(x, shift, scale, eps)
        else:
            y, mean, rstd = lnmod.forward_varlen(x, shift, scale, cu_seqlens, eps)
        ctx.eps = eps
        if save_stats:
            ctx.save_for_backward(x, scale, cu_seqlens, mean, rstd)
        else:                                   # the backward forms them again from x
            ctx.save_for_backward(x, scale, cu_seqlens, None, None)
        return y

    @staticmethod
    def backward(ctx, dy):
        x, scale, cu, mean, rstd = ctx.saved_tensors
        return _ln_backward(dy.contiguous(), x, scale, cu, mean, rstd, ctx.eps) + (None, None, None)


def ln_modulate(x, shift, scale, eps=1e-6, cu_seqlens=None, save_stats=True):
    """y = LayerNorm(x) * (1 + scale) + shift (no affine, fp32 statistics).  save_stats=False keeps
    only x between the passes; the backward then recomputes mean and rstd."""
    host = lnmod.native()
    y = None if host is None else host.ln_modulate(x, shift, scale, cu_seqlens, float(eps), bool(save_stats))
    return _LnModulate.apply(x, shift, scale, cu_seqlens, float(eps), bool(save_stats)) if y is None else y


def _gated_backward(dy, dh, h, u, gate, scale, mean, rstd, cu_seqlens, eps):
    return lnmod._gated_backward(dy, dh, h, u, gate, scale, mean, rstd, cu_seqlens, eps, io_grads=True)


class _GatedLnModulate(torch.autograd.Function):
    """Sec. 4.4 "Gate + Norm": the residual update and the LayerNorm-Modulate after it."""

    @staticmethod
    def forward(ctx, x, u, gate, shift, scale, cu_seqlens, eps):
        _contig(x, u, gate, shift, scale, cu_seqlens)
        h, y, mean, rstd = lnmod.gated_forward(x, u, gate, shift, scale, cu_seqlens, eps)
        ctx.eps = eps
        ctx.save_for_backward(h, u, gate, scale, cu_seqlens, mean, rstd)
        return h, y

    @staticmethod
    def backward(ctx, dh, dy):
        h, u, gate, scale, cu, mean, rstd = ctx.saved_tensors
        return _gated_backward(dy.contiguous(), dh.contiguous(), h, u, gate, scale, mean, rstd, cu,
                               ctx.eps) + (None, None)


def gated_ln_modulate(x, u, gate, shift, scale, eps=1e-6, cu_seqlens=None):
    """h = x + gate * u (returned, it is the new residual stream) and y = LN(h) * (1 + scale) + shift."""
    host = lnmod.native()
    r = None if host is None else host.gated_ln_modulate(x, u, gate, shift, scale, cu_seqlens, float(eps))
    return _GatedLnModulate.apply(x, u, gate, shift, scale, cu_seqlens, float(eps)) if r is None else r


def _qk_backward(dqn, dkn, q, k, wq, wk, rq, rk, eps):
    return lnmod._qknorm_backward(dqn, dkn, q, k, wq, wk, rq, rk, eps, io_grads=True)


class _QkNorm(torch.autograd.Function):
    """Sec. 4.4 fused Q-Norm + K-Norm."""

    @staticmethod
    def forward(ctx, q, k, wq, wk, eps):
        _contig(q, k, wq, wk)
        qn, kn, rq, rk = lnmod.qknorm_forward(q, k, wq, wk, eps)
        ctx.eps = eps
        ctx.save_for_backward(q, k, wq, wk, rq, rk)
        return qn, kn

    @staticmethod
    def backward(ctx, dqn, dkn):
        q, k, wq, wk, rq, rk = ctx.saved_tensors
        return _qk_backward(dqn.contiguous(), dkn.contiguous(), q, k, wq, wk, rq, rk, ctx.eps) + (None,)


def qk_norm(q, k, wq, wk, eps=1e-6):
    """q * rsqrt(mean(q^2) + eps) * wq and the same for k, in one launch."""
    host = lnmod.native()
    r = None if host is None else host.qk_norm(q, k, wq, wk, float(eps))
    return _QkNorm.apply(q, k, wq, wk, float(eps)) if r is None else r
