"""The workloads whose speed this repository cares about, as cases that a
timing program can prepare and run.

A case is a dict of plain values: ``op`` (what is called), ``dtype``, the
domain ``ni, nj, nk`` and the options of that call.  ``prepare`` makes on the
GPU what a program holds before the call (fields, masks, workspaces, a captured
graph), ``run`` is one pass through the public entry points, ``work`` the
bytes and operations that pass cannot do without, ``exact`` its results in 64
bits in plain torch.

Inputs have the distributions of ``paper_2311_08322_amd/inputs.py`` (u in
[0, 1) with its halo, w in [-1, 1], data in [-0.1, 0.1], cotangents in
[-1, 1], coefficient fields in [coeff/2, 3 coeff/2)), drawn on the device.
Fields of the C-ABI calls are the library's own storages; the autograd cases
use the contiguous tensors that their interface takes.  No case tunes: a call
without tuning is what a program does first.
"""
from __future__ import annotations

import numpy as np
import torch

from paper_2311_08322_amd import api, autograd, fields, inputs
from paper_2311_08322_amd.frontend import stencils

DEV = "cuda"
COEFF, DT_DZ = inputs.COEFF, inputs.DT_DZ
DTYPES = {"float64": torch.float64, "float32": torch.float32}


def listed():
    return [
        # one diffusion call on the smallest configuration: the launch and the call itself
        dict(name="hdiff_64x64x16_f64", op="hdiff", dtype="float64", ni=64, nj=64, nk=16, field=False, damping=False),
        # the fused step of the largest configuration, called step by step from a model's time loop
        dict(name="step_512x512x80_f64", op="step", dtype="float64", ni=512, nj=512, nk=80, mask=False),
        # the same in single precision, saving the limiter decisions for a later adjoint
        dict(name="step_mask_512x512x80_f32", op="step", dtype="float32", ni=512, nj=512, nk=80, mask=True),
        # a time loop captured as one graph, periodic boundaries, the middle configuration
        dict(name="loop_256x256x80_f64", op="loop", dtype="float64", ni=256, nj=256, nk=80, steps=8),
        # the step adjoint of the adjoint configuration (4D-Var, sensitivity runs)
        dict(name="adjoint_256x256x80_f64", op="adjoint", dtype="float64", ni=256, nj=256, nk=80),
        # 32 uneven subdomains stepped by one call: the batched configuration
        dict(name="batch32_f64", op="batch", dtype="float64", fields=32, sizes_seed=-1),
        # their adjoint in single precision
        dict(name="batch32_adjoint_f32", op="batch_adjoint", dtype="float32", fields=32, sizes_seed=-1),
        # parameter tuning: forward and backward with gradients to state, forcing, w and the scalar coefficient
        dict(name="train_scalar_256x256x80_f64", op="train", dtype="float64", ni=256, nj=256, nk=80, field=False,
             damping=False),
        # a learned per-point coefficient in the damping form, odd sizes, single precision
        dict(name="train_field_501x403x60_f32", op="train", dtype="float32", ni=501, nj=403, nk=60, field=True,
             damping=True),
        # the generalised diffusion alone with a coefficient field
        dict(name="hdiff_field_384x384x64_f64", op="hdiff", dtype="float64", ni=384, nj=384, nk=64, field=True,
             damping=False),
        # the implicit column solve alone on the longest columns of the batched range, odd sizes
        dict(name="vadv_301x203x137_f64", op="vadv", dtype="float64", ni=301, nj=203, nk=137),
        # the step written in the stencil language: a user's own stencil through the generated kernels
        dict(name="frontend_step_512x512x80_f64", op="frontend", dtype="float64", ni=512, nj=512, nk=80, stencil="step"),
    ]


def _log_int(rng, lo, hi):
    return int(round(float(np.exp(rng.uniform(np.log(lo), np.log(hi))))))


def draw(rng):
    op = rng.choice(["hdiff", "vadv", "step", "loop", "adjoint", "batch", "batch_adjoint", "train", "frontend"])
    c = dict(op=op, dtype=rng.choice(["float64", "float32"]))
    if op in ("batch", "batch_adjoint"):
        most = sum(int(np.prod(d)) for d in inputs.batch_sizes())  # the listed batch's points
        c.update(fields=rng.randint(4, 24), sizes_seed=rng.randint(0, 1 << 20))
        while sum(int(np.prod(d)) for d in _sizes(c)) > most:
            c.update(sizes_seed=rng.randint(0, 1 << 20))
        return c
    ni, nj = _log_int(rng, 16, 512), _log_int(rng, 16, 512)
    nk = _log_int(rng, 8, 137)
    while ni * nj * nk > 512 * 512 * 80:
        nk = nk * 3 // 4
    c.update(ni=ni, nj=nj, nk=nk)
    if op in ("hdiff", "train"):
        c.update(field=rng.random() < 0.5, damping=rng.random() < 0.5)
    elif op == "step":
        c.update(mask=rng.random() < 0.5)
    elif op == "loop":
        # binary32 states drift apart by whole limiter decisions over many steps
        c.update(dtype="float64", steps=2 * rng.randint(1, 8))
    elif op == "frontend":
        c.update(stencil=rng.choice(["step", "hdiff", "vadv"]))
    return c


# ------------------------------------------------------------------ inputs
def _sizes(case):
    """The (ni, nj, nk) of a case's fields."""
    if "fields" not in case:
        return [(case["ni"], case["nj"], case["nk"])]
    if case["sizes_seed"] < 0:
        return inputs.batch_sizes(case["fields"])
    r = np.random.default_rng(case["sizes_seed"])
    return [tuple(int(r.integers(lo, hi, endpoint=True)) for lo, hi in inputs.BATCH_RANGE) for _ in range(case["fields"])]


def _draw_inputs(dom, dtype, g, xbar=False, kappa=False):
    """Contiguous u (padded), data, w (nk + 1 levels) and, when asked, a
    cotangent and a coefficient field."""
    ni, nj, nk = dom

    def uniform(shape, lo, hi):
        return torch.empty(shape, dtype=dtype, device=DEV).uniform_(lo, hi, generator=g)

    r = dict(u=uniform((nk, nj + 4, ni + 4), 0.0, 1.0), data=uniform((nk, nj, ni), -0.1, 0.1),
             w=uniform((nk + 1, nj, ni), -1.0, 1.0))
    if xbar:
        r["xbar"] = uniform((nk, nj, ni), -1.0, 1.0)
    if kappa:
        r["kappa"] = uniform((nk, nj, ni), 0.5 * COEFF, 1.5 * COEFF)
    return r


def _all_inputs(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    dt = DTYPES[case["dtype"]]
    xbar = case["op"] in ("adjoint", "batch_adjoint", "train")
    return [_draw_inputs(dom, dt, g, xbar, case.get("field", False)) for dom in _sizes(case)]


def _padded_field(t):
    nk, nj, ni = t.shape
    f = fields.alloc(ni - 4, nj - 4, nk, t.dtype, DEV, fill=0.0)
    fields.padded(f, ni - 4, nj - 4, nk).copy_(t)
    return f


def _interior_field(t):
    nk, nj, ni = t.shape
    f = fields.alloc(ni, nj, nk, t.dtype, DEV, halo=0, fill=0.0)
    fields.interior(f, ni, nj, nk).copy_(t)
    return f


def _empty_padded(dom, dt):
    return fields.alloc(*dom, dt, DEV, fill=0.0)


def _empty_interior(dom, dt):
    return fields.alloc(*dom, dt, DEV, halo=0, fill=0.0)


def _forward_mask(x, dom):
    """The limiter decisions of the forward step on these inputs."""
    mask = fields.mask_tensor(dom, DEV)
    out = _empty_interior(dom, x["u"].dtype)
    api.stencil_step(_padded_field(x["u"]), _interior_field(x["data"]), _interior_field(x["w"]), out, dom, COEFF,
                     DT_DZ, mask=mask)
    return mask


# ------------------------------------------------------------------ prepare
def prepare(case, seed):
    op, dt = case["op"], DTYPES[case["dtype"]]
    xs = _all_inputs(case, seed)
    doms = _sizes(case)
    dom, x = doms[0], xs[0]
    ni, nj, nk = dom
    s = dict(op=op, dom=dom)
    if op == "hdiff":
        out = _empty_interior(dom, dt)
        s.update(u=_padded_field(x["u"]), out=out, result=fields.interior(out, *dom), opts=None)
        if case["field"] or case["damping"]:
            s["opts"] = api.Options(hdiff_form=api.HDIFF_DAMPING if case["damping"] else api.HDIFF_STATED,
                                    coeff_field=_interior_field(x["kappa"]) if case["field"] else None)
    elif op == "vadv":
        out = _empty_interior(dom, dt)
        s.update(u=_interior_field(x["u"][:, 2:-2, 2:-2]), data=_interior_field(x["data"]), w=_interior_field(x["w"]),
                 out=out, result=fields.interior(out, *dom))
    elif op == "step":
        out = _empty_interior(dom, dt)
        s.update(u=_padded_field(x["u"]), data=_interior_field(x["data"]), w=_interior_field(x["w"]), out=out,
                 mask=fields.mask_tensor(dom, DEV) if case["mask"] else None)
        s["result"] = [fields.interior(out, *dom)] + ([s["mask"]] if case["mask"] else [])
    elif op == "loop":
        ua, ub = _padded_field(x["u"]), _padded_field(x["u"])
        s.update(u=ua, ub=ub, data=_interior_field(x["data"]), w=_interior_field(x["w"]),
                 opts=api.Options(boundary=api.BOUNDARY_PERIODIC), side=torch.cuda.Stream(),
                 result=fields.padded(ua, *dom))
        torch.cuda.synchronize()
        s["graph"] = api.stencil_graph_capture_steps(case["steps"], ua, ub, s["data"], s["w"], dom, COEFF, DT_DZ,
                                                     opts=s["opts"], stream=s["side"])
    elif op == "adjoint":
        ub, db = _empty_padded(dom, dt), _empty_interior(dom, dt)
        s.update(xbar=_interior_field(x["xbar"]), w=_interior_field(x["w"]), mask=_forward_mask(x, dom), ubar=ub,
                 dbar=db, result=[fields.padded(ub, *dom), fields.interior(db, *dom)])
    elif op == "batch":
        items = [dict(u=_padded_field(y["u"]), data=_interior_field(y["data"]), w=_interior_field(y["w"]),
                      out=_empty_interior(d, dt), domain=d, coeff=COEFF, dt_dz=DT_DZ) for y, d in zip(xs, doms)]
        n = api.stencil_batch_workspace_bytes(dt, items)
        s.update(dtype=dt, items=items, ws=torch.empty(n, dtype=torch.uint8, device=DEV),
                 result=[fields.interior(it["out"], *it["domain"]) for it in items])
    elif op == "batch_adjoint":
        items = [dict(x_bar=_interior_field(y["xbar"]), w=_interior_field(y["w"]), mask=_forward_mask(y, d),
                      u_bar=_empty_padded(d, dt), data_bar=_empty_interior(d, dt), domain=d, coeff=COEFF, dt_dz=DT_DZ)
                 for y, d in zip(xs, doms)]
        n = api.stencil_batch_adjoint_workspace_bytes(dt, items)
        s.update(dtype=dt, items=items, ws=torch.empty(n, dtype=torch.uint8, device=DEV),
                 result=[v for it in items for v in (fields.padded(it["u_bar"], *it["domain"]),
                                                     fields.interior(it["data_bar"], *it["domain"]))])
    elif op == "train":
        c = x["kappa"] if case["field"] else torch.tensor(COEFF, dtype=dt, device=DEV)
        s.update(leaves=[x["u"].requires_grad_(), x["data"].requires_grad_(), x["w"].requires_grad_(),
                         c.requires_grad_()], xbar=x["xbar"], damping=case["damping"])
    elif op == "frontend":
        fn = stencils.ALL[case["stencil"]]
        out = _empty_interior(dom, dt)
        u = _interior_field(x["u"][:, 2:-2, 2:-2]) if case["stencil"] == "vadv" else _padded_field(x["u"])
        args = [u] + ([] if case["stencil"] == "hdiff" else [_interior_field(x["data"]), _interior_field(x["w"])]) + [out]
        scalars = {k: v for k, v in (("coeff", COEFF), ("dt_dz", DT_DZ)) if k in fn.definition.scalars}
        s.update(fn=fn, args=args, scalars=scalars, result=fields.interior(out, *dom))
        fn.build(case["dtype"])  # the cached library, loaded once by a program
    return s


# ------------------------------------------------------------------ run
def run(s):
    op, dom = s["op"], s["dom"]
    if op == "hdiff":
        api.stencil_hdiff(s["u"], s["out"], dom, COEFF, opts=s["opts"])
    elif op == "vadv":
        api.stencil_vadv(s["u"], s["data"], s["w"], s["out"], dom, DT_DZ)
    elif op == "step":
        api.stencil_step(s["u"], s["data"], s["w"], s["out"], dom, COEFF, DT_DZ, mask=s["mask"])
    elif op == "loop":
        api.stencil_graph_launch(s["graph"])
    elif op == "adjoint":
        api.stencil_step_adjoint(s["xbar"], s["w"], s["mask"], s["ubar"], s["dbar"], dom, COEFF, DT_DZ)
    elif op == "batch":
        api.stencil_step_batched(s["dtype"], s["items"], s["ws"])
    elif op == "batch_adjoint":
        api.stencil_step_adjoint_batched(s["dtype"], s["items"], s["ws"])
    elif op == "train":
        out = autograd.step(*s["leaves"], dt_dz=DT_DZ, damping=s["damping"])
        return [out.detach(), *torch.autograd.grad(out, s["leaves"], s["xbar"])]
    elif op == "frontend":
        s["fn"](*s["args"], domain=dom, **s["scalars"])
    return s["result"]


# ------------------------------------------------------------------ work
def work(case):
    size = 8 if case["dtype"] == "float64" else 4
    op = case["op"]
    b = f = 0
    for ni, nj, nk in _sizes(case):
        n, pad = ni * nj * nk, (ni + 4) * (nj + 4) * nk
        w = (nk - 1) * ni * nj  # staggered levels 1 .. nk-1 enter the solve
        mask = n // 4           # two decisions a point
        diffuse, solve = 30 * n, 15 * n
        if op == "hdiff" or case.get("stencil") == "hdiff":
            b += size * (pad + n + (n if case.get("field") else 0))
            f += diffuse
        elif op == "vadv" or case.get("stencil") == "vadv":
            b += size * (3 * n + w)
            f += solve
        elif op in ("step", "batch") or op == "frontend":
            b += size * (pad + 2 * n + w) + (mask if case.get("mask") else 0)
            f += diffuse + solve
        elif op == "loop":
            b += case["steps"] * size * (2 * pad + n + w)
            f += case["steps"] * (diffuse + solve)
        elif op in ("adjoint", "batch_adjoint"):
            b += size * (2 * n + w + pad) + mask
            f += diffuse + solve
        elif op == "train":
            b += size * (2 * pad + 4 * n + 2 * w + (2 * n if case["field"] else 0))
            f += 3 * (diffuse + solve)
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------ exact
def _lap(u):
    return 4.0 * u[:, 1:-1, 1:-1] - ((u[:, 1:-1, :-2] + u[:, 1:-1, 2:]) + (u[:, :-2, 1:-1] + u[:, 2:, 1:-1]))


def _fluxes(u, sign):
    """x fluxes on [-1, ni) x [0, nj), y fluxes on [0, ni) x [-1, nj), and the
    gradients of u that limit them."""
    lap = sign * _lap(u)
    fx, fy = lap[:, 1:-1, 1:] - lap[:, 1:-1, :-1], lap[:, 1:, 1:-1] - lap[:, :-1, 1:-1]
    return fx, fy, u[:, 2:-2, 2:-1] - u[:, 2:-2, 1:-2], u[:, 2:-1, 2:-2] - u[:, 1:-2, 2:-2]


def _kept(u, damping):
    """The limiter's decisions, taken in the fields' own precision."""
    fx, fy, gx, gy = _fluxes(u, -1.0 if damping else 1.0)
    return ~(fx * gx > 0), ~(fy * gy > 0)


def _hdiff(u, coeff, damping, kept):
    fx, fy, _, _ = _fluxes(u, -1.0 if damping else 1.0)
    fx, fy = fx * kept[0], fy * kept[1]
    return u[:, 2:-2, 2:-2] - coeff * ((fx[:, :, 1:] - fx[:, :, :-1]) + (fy[:, 1:] - fy[:, :-1]))


def _solve(d, w):
    nk, r4 = d.shape[0], 0.25 * DT_DZ
    cp, dp = [], []
    for k in range(nk):
        c = r4 * w[k + 1] if k < nk - 1 else torch.zeros_like(w[0])
        if k == 0:
            m = 1.0 + c.abs()
            cp.append(c / m)
            dp.append(d[0] / m)
        else:
            a = -r4 * w[k]
            m = 1.0 + a.abs() + c.abs() - a * cp[-1]
            cp.append(c / m)
            dp.append((d[k] - a * dp[-1]) / m)
    x = [dp[-1]]
    for k in range(nk - 2, -1, -1):
        x.append(dp[k] - cp[k] * x[-1])
    return torch.stack(x[::-1])


def _coefficient(x):
    """The coefficient as the call rounds it to the fields' type, in 64 bits."""
    return x["kappa"].double() if "kappa" in x else torch.tensor(COEFF, dtype=x["u"].dtype, device=DEV).double()


def _step_gradients(x, damping, wanted):
    kept = _kept(x["u"], damping)
    leaves = dict(u=x["u"].double(), data=x["data"].double(), w=x["w"].double(), coeff=_coefficient(x))
    for v in leaves.values():
        v.requires_grad_()
    out = _solve(_hdiff(leaves["u"], leaves["coeff"], damping, kept) + leaves["data"], leaves["w"])
    return out.detach(), torch.autograd.grad(out, [leaves[k] for k in wanted], x["xbar"].double())


def exact(case, seed):
    op = case["op"]
    res = []
    for x in _all_inputs(case, seed):
        if op in ("hdiff", "step", "batch") or case.get("stencil") in ("hdiff", "step"):
            damping = case.get("damping", False)
            v = _hdiff(x["u"].double(), _coefficient(x), damping, _kept(x["u"], damping))
            if op in ("step", "batch") or case.get("stencil") == "step":
                v = _solve(v + x["data"].double(), x["w"].double())
            res.append(v)
        elif op == "vadv" or case.get("stencil") == "vadv":
            res.append(_solve(x["u"][:, 2:-2, 2:-2].double() + x["data"].double(), x["w"].double()))
        elif op == "loop":
            u = x["u"]
            for _ in range(case["steps"]):
                v = _solve(_hdiff(u, COEFF, False, _kept(u, False)) + x["data"], x["w"])
                u = torch.nn.functional.pad(v[:, None], (2, 2, 2, 2), mode="circular")[:, 0]
            res.append(u)
        elif op in ("adjoint", "batch_adjoint"):
            res += _step_gradients(x, False, ("u", "data"))[1]
        elif op == "train":
            out, grads = _step_gradients(x, case["damping"], ("u", "data", "w", "coeff"))
            res += [out, *grads]
    if op == "step" and case["mask"]:
        return [res[0], None]  # the packed decisions have no 64-bit value
    return res[0] if op in ("hdiff", "vadv", "loop", "frontend") else res
