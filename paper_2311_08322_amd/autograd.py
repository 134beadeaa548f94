"""torch.autograd wrappers: the forward calls the fused HIP step (saving the
limiter mask), the backward calls the hand-written adjoint kernels.

Tensors use the canonical contiguous layouts (k, j, i):
  u       (nk, nj+4, ni+4)  -- domain plus its 2-point halo
  data    (nk, nj, ni)
  w       (nk+1, nj, ni)    -- staggered levels
  coeff   a float, a 0-d tensor, or a per-point field (nk, nj, ni)
Outputs are the new interior values (nk, nj, ni).  Gradients of the step
flow to u (over its halo as well), data, w and a tensor coeff (scalar or
field); the step is differentiated almost everywhere, with the limiter
decisions of the forward pass held fixed (and d|t|/dt = 0 at t = 0 in the
diagonal of T).  `damping=True` selects the damping form of the diffusion.
"""
from __future__ import annotations

import torch

from . import api

HALO = 2


def _f(t: torch.Tensor, halo: int) -> api.Field:
    return api.Field(t, (halo, halo, 0))


def _dims(data: torch.Tensor):
    nk, nj, ni = data.shape
    return ni, nj, nk


def _opts(coeff, damping):
    """Options of the generalised diffusion: the damping form and, for a
    coefficient tensor with dimensions, the per-point field."""
    field = torch.is_tensor(coeff) and coeff.dim() == 3
    return api.Options(hdiff_form=api.HDIFF_DAMPING if damping else api.HDIFF_STATED,
                       coeff_field=_f(coeff, 0) if field else None), field


# longest columns of the step that reads its coefficient from device memory
_DEV_COEFF_NK = {torch.float64: 144, torch.float32: 160}


def _dense_call(like, shapes, *tensors):
    """Whether the tensors are what the training calls take: non-empty contiguous
    device tensors of one floating type on one device, in the canonical shapes
    (other calls go through fields, which also serve larger tensors)."""
    return (like.is_cuda and like.dtype in _DEV_COEFF_NK and like.numel() > 0 and
            all(t.shape == s and t.dtype == like.dtype and t.device == like.device for t, s in zip(tensors, shapes)))


def _forward_dense(ctx, u, data, w, out, kap, coeff, dom, dt_dz, damping):
    """The forward call.  A scalar coefficient tensor on the fields' device is
    read by the kernel, which leaves its value behind the mask for the backward:
    no copy to the host, and later changes of the tensor do not reach it."""
    n = api.stencil_mask_bytes(dom)
    mask = torch.empty(n + 256, dtype=torch.uint8, device=out.device)
    dev = None
    if kap is None and torch.is_tensor(coeff) and coeff.device == out.device and coeff.dtype in _DEV_COEFF_NK and (
            coeff.numel() == 1 and (w is None or dom[2] <= _DEV_COEFF_NK[out.dtype])):
        dev = coeff.detach()
        dev.record_stream(torch.cuda.current_stream())  # the kernel may read it after the caller drops it
    c = 0.0 if kap is not None or dev is not None else float(coeff)
    ctx.copy_at = n if dev is not None else None
    api.stencil_train_forward(u, data, w, out, mask, kap, c, dev, mask.data_ptr() + n if dev is not None else None,
                              dom, float(dt_dz), api.HDIFF_DAMPING if damping else api.HDIFF_STATED)
    return mask, c


def _backward_dense(ctx, xbar, mask, u, w, out, kap, want_w, want_c):
    """One call for every gradient: (u_bar, data_bar, w_bar, coeff_bar)."""
    ni, nj, nk = ctx.dom
    dt, dev = xbar.dtype, xbar.device
    ubar = torch.empty((nk, nj + 2 * HALO, ni + 2 * HALO), dtype=dt, device=dev)
    dbar = torch.empty_like(xbar) if w is not None else None
    wbar = torch.empty_like(w) if want_w else None
    kbar = torch.empty_like(xbar) if want_c and ctx.field else None
    cbar = ws = None
    if want_c and not ctx.field:
        cbar = torch.empty((), dtype=dt, device=dev)
        ws = torch.empty(api.stencil_param_workspace_bytes(dt, ctx.dom), dtype=torch.uint8, device=dev)
    api.stencil_train_backward(xbar, mask, u, w, out, kap, ctx.coeff,
                               None if ctx.copy_at is None else mask.data_ptr() + ctx.copy_at, ubar, dbar, wbar, kbar,
                               cbar, ws, ctx.dom, float(ctx.dt_dz),
                               api.HDIFF_DAMPING if ctx.damping else api.HDIFF_STATED)
    return ubar, dbar, wbar, kbar if kbar is not None else cbar


class StencilStep(torch.autograd.Function):
    """x = vadv(hdiff(u), data, w): one fused time step.  coeff may be a
    float, a 0-d tensor or a per-point field; gradients flow to u, data, w
    and a tensor coeff."""

    @staticmethod
    def forward(ctx, u, data, w, coeff, dt_dz: float, damping: bool = False):
        u, data, w = u.contiguous(), data.contiguous(), w.contiguous()
        ni, nj, nk = _dims(data)
        dom = (ni, nj, nk)
        if torch.is_tensor(coeff) and coeff.dim() == 3:
            coeff = coeff.contiguous()
        field = torch.is_tensor(coeff) and coeff.dim() == 3
        out = torch.empty_like(data)
        ctx.dense = _dense_call(data, ((nk, nj + 2 * HALO, ni + 2 * HALO), (nk + 1, nj, ni), data.shape), u, w,
                                *([coeff] if field else []))
        if ctx.dense:
            mask, c = _forward_dense(ctx, u, data, w, out, coeff if field else None, coeff, dom, dt_dz, damping)
        else:
            opts, _ = _opts(coeff, damping)
            c = 0.0 if field else float(coeff)
            mask = torch.empty(max(api.stencil_mask_bytes(dom), 1), dtype=torch.uint8, device=u.device)
            api.stencil_step(_f(u, HALO), _f(data, 0), _f(w, 0), _f(out, 0), dom, c, dt_dz, mask=mask, opts=opts)
        ctx.params = ctx.needs_input_grad[2] or (torch.is_tensor(coeff) and ctx.needs_input_grad[3])
        # the parameter gradients need the step's input and output
        ctx.save_for_backward(w, mask, u if ctx.params else None, out if ctx.params else None,
                              coeff if field else None)
        ctx.coeff, ctx.dt_dz, ctx.dom, ctx.damping, ctx.field = c, dt_dz, dom, damping, field
        ctx.coeff_tensor = torch.is_tensor(coeff)
        return out

    @staticmethod
    def backward(ctx, xbar):
        w, mask, u, out, kap = ctx.saved_tensors
        ni, nj, nk = ctx.dom
        xbar = xbar.contiguous()
        if ctx.dense:
            ubar, dbar, wbar, cbar = _backward_dense(ctx, xbar, mask, u, w, out, kap, ctx.needs_input_grad[2],
                                                     ctx.coeff_tensor and ctx.needs_input_grad[3])
            return ubar, dbar, wbar, cbar, None, None
        opts, _ = _opts(kap if ctx.field else ctx.coeff, ctx.damping)
        ubar = torch.empty((nk, nj + 2 * HALO, ni + 2 * HALO), dtype=xbar.dtype, device=xbar.device)
        dbar = torch.empty_like(xbar)
        api.stencil_step_adjoint(_f(xbar, 0), _f(w, 0), mask, _f(ubar, HALO), _f(dbar, 0), ctx.dom, ctx.coeff,
                                 ctx.dt_dz, opts=opts)
        wbar = cbar = None
        if ctx.params:
            want_w = ctx.needs_input_grad[2]
            want_c = ctx.coeff_tensor and ctx.needs_input_grad[3]
            if want_c and ctx.field:
                kb = torch.empty_like(xbar)
                api.stencil_coeff_field_adjoint(_f(u, HALO), _f(dbar, 0), _f(kb, 0), ctx.dom, opts=opts)
                cbar = kb
            want_scalar = want_c and not ctx.field
            if want_w or want_scalar:
                wb = torch.empty_like(w) if want_w else None
                cb = torch.zeros(1, dtype=torch.float64, device=xbar.device) if want_scalar else None
                n = api.stencil_param_workspace_bytes(xbar.dtype, ctx.dom) if want_scalar else 0
                ws = torch.empty(n, dtype=torch.uint8, device=xbar.device) if n else None
                api.stencil_step_param_adjoint(_f(u, HALO), _f(w, 0), _f(out, 0), _f(dbar, 0),
                                               _f(wb, 0) if want_w else None, cb, ctx.dom, ctx.dt_dz, ws=ws,
                                               dtype=xbar.dtype, opts=opts)
                wbar = wb
                if want_scalar:
                    cbar = cb.reshape(()).to(xbar.dtype)
        return ubar, dbar, wbar, cbar, None, None


class HDiff(torch.autograd.Function):
    """out = hdiff(u) on the interior; coeff a float, a 0-d tensor or a
    per-point field, with gradients to u and a tensor coeff."""

    @staticmethod
    def forward(ctx, u, coeff, damping: bool = False):
        u = u.contiguous()
        nk, Nj, Ni = u.shape
        dom = (Ni - 2 * HALO, Nj - 2 * HALO, nk)
        if torch.is_tensor(coeff) and coeff.dim() == 3:
            coeff = coeff.contiguous()
        field = torch.is_tensor(coeff) and coeff.dim() == 3
        out = torch.empty((nk, dom[1], dom[0]), dtype=u.dtype, device=u.device)
        ctx.dense = _dense_call(out, (out.shape,), *([coeff] if field else []))
        if ctx.dense:
            mask, c = _forward_dense(ctx, u, None, None, out, coeff if field else None, coeff, dom, 0.5, damping)
        else:
            opts, _ = _opts(coeff, damping)
            c = 0.0 if field else float(coeff)
            mask = torch.empty(max(api.stencil_mask_bytes(dom), 1), dtype=torch.uint8, device=u.device)
            api.stencil_hdiff(_f(u, HALO), _f(out, 0), dom, c, mask=mask, opts=opts)
        want_c = torch.is_tensor(coeff) and ctx.needs_input_grad[1]
        ctx.save_for_backward(mask, u if want_c else None, coeff if field else None)
        ctx.coeff, ctx.dom, ctx.damping, ctx.field, ctx.want_c = c, dom, damping, field, want_c
        ctx.dt_dz = 0.5  # the diffusion has none
        return out

    @staticmethod
    def backward(ctx, obar):
        mask, u, kap = ctx.saved_tensors
        ni, nj, nk = ctx.dom
        obar = obar.contiguous()
        if ctx.dense:
            ubar, _, _, cbar = _backward_dense(ctx, obar, mask, u, None, None, kap, False, ctx.want_c)
            return ubar, cbar, None
        opts, _ = _opts(kap if ctx.field else ctx.coeff, ctx.damping)
        ubar = torch.empty((nk, nj + 2 * HALO, ni + 2 * HALO), dtype=obar.dtype, device=obar.device)
        api.stencil_hdiff_adjoint(_f(obar, 0), mask, _f(ubar, HALO), ctx.dom, ctx.coeff, opts=opts)
        cbar = None
        if ctx.want_c and ctx.field:
            kb = torch.empty_like(obar)
            api.stencil_coeff_field_adjoint(_f(u, HALO), _f(obar, 0), _f(kb, 0), ctx.dom, opts=opts)
            cbar = kb
        elif ctx.want_c:  # the scalar: -sum obar * D(u), the parameter adjoint with lambda = obar
            cb = torch.zeros(1, dtype=torch.float64, device=obar.device)
            n = api.stencil_param_workspace_bytes(obar.dtype, ctx.dom)
            ws = torch.empty(n, dtype=torch.uint8, device=obar.device) if n else None
            api.stencil_step_param_adjoint(_f(u, HALO), None, None, _f(obar, 0), None, cb, ctx.dom, 0.5, ws=ws,
                                           dtype=obar.dtype, opts=opts)
            cbar = cb.reshape(()).to(obar.dtype)
        return ubar, cbar, None


class VAdv(torch.autograd.Function):
    """x = T(w)^{-1} (u + data) per column."""

    @staticmethod
    def forward(ctx, u, data, w, dt_dz: float):
        u, data, w = u.contiguous(), data.contiguous(), w.contiguous()
        dom = _dims(data)
        out = torch.empty_like(data)
        api.stencil_vadv(_f(u, 0), _f(data, 0), _f(w, 0), _f(out, 0), dom, dt_dz)
        ctx.save_for_backward(w)
        ctx.dt_dz, ctx.dom = dt_dz, dom
        return out

    @staticmethod
    def backward(ctx, xbar):
        (w,) = ctx.saved_tensors
        xbar = xbar.contiguous()
        lam = torch.empty_like(xbar)
        api.stencil_vadv_adjoint(_f(xbar, 0), _f(w, 0), _f(lam, 0), ctx.dom, ctx.dt_dz)
        return lam, lam, None, None


def step(u, data, w, coeff=0.025, dt_dz=0.5, damping=False):
    return StencilStep.apply(u, data, w, coeff, dt_dz, damping)


def hdiff(u, coeff=0.025, damping=False):
    return HDiff.apply(u, coeff, damping)


def vadv(u, data, w, dt_dz=0.5):
    return VAdv.apply(u, data, w, dt_dz)
