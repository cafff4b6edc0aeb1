"""torch.autograd functions over the HIP kernels, for DPD coefficient
adaptation through a fixed memory-polynomial PA model.

Gradients follow torch's convention for complex tensors, dL/dRe z + i dL/dIm z,
which is the convention of the library's adjoint kernels.

    u = DPDFunction.apply(x, h, r)        # predistortion, learnable h
    v = PAFunction.apply(u, a)            # fixed PA: v = sum a[k][q] |u|^(2k) u (delay q)
    loss = (v - x).abs().pow(2).sum()
    loss.backward()                        # h.grad from the hand-written adjoints

Every tensor here is complex64 on the GPU; all arithmetic of the forward and
backward passes runs in libdfhip.so on torch's current stream.
"""
from __future__ import annotations

import torch

from . import dfhip as D


def _stream():
    return torch.cuda.current_stream()


def _forward(x, ctrl, h, y, r, hist):
    """y = DPD_h(x) with torch's allocations as scratch (cached, and ordered on
    torch's stream); returns the firings' tables, None without ctrl."""
    D.check_dpd_tensors(x, ctrl, h, y, r)
    (S, L), (B, M) = x.shape, h.shape
    tables = None
    if ctrl is not None:
        tables = torch.empty(max(D.df_dpd_tables_bytes(S, L, r, B), 8), dtype=torch.uint8, device=x.device)
    work = torch.empty(max(D.df_dpd_forward_work_bytes(S, L, r, B, M, ctrl is not None), 8), dtype=torch.uint8,
                       device=x.device)
    D.df_dpd_forward_work(x, ctrl, h, y, r, tables, work, hist, stream=_stream())
    return tables


class DPDFunction(torch.autograd.Function):
    """y = DPD_h(x) for x [S, L], h [B, M]; ctrl [S, L/r] int32 or None (all
    branches active).  Backward: coefficient adjoint only (x is data)."""

    @staticmethod
    def forward(ctx, x, h, r: int, ctrl=None, hist: int = D.DF_HIST_BRANCH):
        x = x.contiguous()
        hc = h.detach().contiguous()
        y = torch.empty_like(x)
        tables = _forward(x, ctrl, hc, y, r, hist)
        none = torch.empty(0)
        # the tables are the control tokens as the backward needs them; the
        # tokens are saved too, so that a change in between is an error
        ctx.save_for_backward(x, none if ctrl is None else ctrl, none if tables is None else tables)
        ctx.has_ctrl = tables is not None
        ctx.r, ctx.hshape = r, h.shape
        return y

    @staticmethod
    def backward(ctx, gy):
        x, _, tables = ctx.saved_tensors
        B, M = ctx.hshape
        S, L = x.shape
        grad_h = None
        if ctx.needs_input_grad[1]:
            grad_h = torch.empty((B, M), dtype=torch.complex64, device=x.device)
            nb = D.df_dpd_coeff_adjoint_work_bytes(S, L, ctx.r, B, M)
            work = torch.empty(max(nb, 8), dtype=torch.uint8, device=x.device)
            if ctx.has_ctrl:
                D.df_dpd_coeff_adjoint_tables(x, tables, gy.contiguous(), grad_h, ctx.r, work, stream=_stream())
            else:
                D.df_dpd_coeff_adjoint(x, None, gy.contiguous(), grad_h, ctx.r, work, stream=_stream())
        return None, grad_h, None, None, None


class PAFunction(torch.autograd.Function):
    """v = PA_a(u): memory polynomial with fixed coefficients a [K, Q]
    (orders 1, 3, .., 2K-1; delays 0..Q-1), evaluated by the predistortion
    kernel with all K branches active.  Backward: input adjoint."""

    @staticmethod
    def forward(ctx, u, a):
        u = u.contiguous()
        a = a.detach().contiguous()
        v = torch.empty_like(u)
        S, L = u.shape
        _forward(u, None, a, v, L, D.DF_HIST_BRANCH)
        ctx.save_for_backward(u, a)
        return v

    @staticmethod
    def backward(ctx, gv):
        u, a = ctx.saved_tensors
        gu = torch.empty_like(u)
        D.df_mp_input_adjoint(u, a, gv.contiguous(), gu, stream=_stream())
        return gu, None


class PALossFunction(torch.autograd.Function):
    """sum |PA_a(u) - x|^2 for fixed a and x, and its gradient for u: the
    model, the error and the sum in one kernel, and the backward reads the
    stored error (the same as PAFunction followed by torch's arithmetic, which
    makes about twenty passes over the signals)."""

    @staticmethod
    def forward(ctx, u, a, x):
        u, a, x = u.contiguous(), a.detach().contiguous(), x.contiguous()
        e = torch.empty_like(u) if ctx.needs_input_grad[0] else None
        loss = torch.empty((), dtype=torch.float32, device=u.device)
        work = torch.empty(D.df_mp_loss_work_bytes(), dtype=torch.uint8, device=u.device)
        D.df_mp_loss(u, a, x, e, loss, work, stream=_stream())
        if e is not None:
            ctx.save_for_backward(u, a, e)
        return loss

    @staticmethod
    def backward(ctx, gloss):
        if not ctx.needs_input_grad[0]:          # only a or x asks, and both are fixed
            return None, None, None
        u, a, e = ctx.saved_tensors
        gu = torch.empty_like(u)
        D.df_mp_loss_adjoint(u, a, e, gloss.contiguous(), gu, stream=_stream())
        return gu, None, None


def adaptation_loss(x, h, a, r):
    """L = sum |PA(DPD_h(x)) - x|^2."""
    u = DPDFunction.apply(x, h, r)
    if not x.requires_grad:
        return PALossFunction.apply(u, a, x)
    e = PAFunction.apply(u, a) - x               # x is a variable too: torch differentiates the error
    return (e.real * e.real + e.imag * e.imag).sum()
