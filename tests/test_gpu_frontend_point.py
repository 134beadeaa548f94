"""Generated kernels evaluated point by point: stencils with offsets of
temporaries, branches, partial intervals, vertical offsets and a pair of
opposite sweeps, at column lengths on both sides of what the stash between the
sweeps holds in registers, in LDS and in the workspace.  The reference is the
same arithmetic in NumPy in the fields' type, operation for operation, so the
values are equal bit for bit."""
import numpy as np
import pytest
import torch

from paper_2311_08322_amd import fields
from paper_2311_08322_amd.frontend import BACKWARD, FORWARD, PARALLEL, Field, computation, interval, stencil
from paper_2311_08322_amd.frontend import hipgen

DTYPES = [torch.float64, torch.float32]
IDS = ["f64", "f32"]


@stencil
def mirror(u: Field, v: Field, out: Field, total: Field, *, alpha: float):
    with computation(PARALLEL), interval(...):
        s = u[1, 0, 0] + u[-1, 0, 0]
        g = s[0, 1, 0] - alpha * s
        if g > 0.0:
            h = g * 0.5
        else:
            h = g + u[0, -1, 0]
    with computation(PARALLEL):
        with interval(0, 2):
            q = v * 2.0
        with interval(2, None):
            q = v - v[0, 0, -1]
    with computation(BACKWARD):
        with interval(-1, None):
            e = q / (2.0 + abs(h))
            f = h
        with interval(0, -1):
            e = q / (2.0 + abs(e[0, 0, 1]))
            f = (h - 0.25 * f[0, 0, 1]) + e
    with computation(FORWARD):
        with interval(0, 1):
            out = f + v
            total = e
        with interval(1, None):
            out = (f - e * out[0, 0, -1]) + v[0, 0, -1]
            total = total[0, 0, -1] + e


@stencil
def pair(u: Field, v: Field, out: Field):
    with computation(PARALLEL):
        with interval(0, -1):
            t = u[1, 0, 1] - u[-1, 0, 0]
            out = t * v[0, 2, 0] + v
        with interval(-1, None):
            out = u * 1.0


@stencil
def rough(u: Field, out: Field):
    with computation(PARALLEL), interval(...):
        t = sqrt(u * u + 1.0)  # noqa: F821 (a builtin of the language)
        out = t[1, 0, 0] - t[0, -1, 0]


def _mirror(u, v, alpha):
    """u has a halo of two points; v and the results are interior."""
    t = u.dtype.type
    nk = v.shape[0]

    def at(a, di, dj):
        return a[:, 2 + dj:a.shape[1] - 2 + dj, 2 + di:a.shape[2] - 2 + di]
    s, s_n = at(u, 1, 0) + at(u, -1, 0), at(u, 1, 1) + at(u, -1, 1)
    g = s_n - t(alpha) * s
    h = np.where(g > 0, g * t(0.5), g + at(u, 0, -1))
    q = v * t(2)
    q[2:] = v[2:] - v[1:-1]
    e, f, out, total = (np.empty_like(v) for _ in range(4))
    for k in range(nk - 1, -1, -1):
        if k == nk - 1:
            e[k], f[k] = q[k] / (t(2) + np.abs(h[k])), h[k]
        else:
            e[k] = q[k] / (t(2) + np.abs(e[k + 1]))
            f[k] = (h[k] - t(0.25) * f[k + 1]) + e[k]
    for k in range(nk):
        out[k] = f[k] + v[k] if k == 0 else (f[k] - e[k] * out[k - 1]) + v[k - 1]
        total[k] = e[k] if k == 0 else total[k - 1] + e[k]
    return out, total


def _plan(st, dtype):
    return hipgen._Gen(st.plan, str(dtype).split(".")[-1], "x").point


def test_plans():
    """The first two take the point form, the factors of the sweeps stashed; a
    square root read at two offsets keeps its LDS stage."""
    assert not _plan(rough, torch.float64)
    assert list(_plan(mirror, torch.float64)) == [0] and _plan(mirror, torch.float64)[0].stash == ["e", "f"]
    assert list(_plan(pair, torch.float32)) == [0] and not _plan(pair, torch.float32)[0].stash


def _levels(dtype):
    _, R, NL = _plan(mirror, dtype)[0]._sizes()
    return [1, 2, 3, R - 1, R, R + 1, R + NL - 1, R + NL, R + NL + 1, R + NL + 5, R + NL + 31]


@pytest.mark.gpu
@pytest.mark.parametrize("at", range(11))
@pytest.mark.parametrize("dtype", DTYPES, ids=IDS)
def test_mirror(dtype, at):
    nk = _levels(dtype)[at]
    for ni, nj in ((67, 5), (1, 1), (64, 8)):
        print(f"mirror {ni}x{nj}x{nk} {dtype}", flush=True)
        r = np.random.default_rng(1000 + nk)
        npd = np.float64 if dtype == torch.float64 else np.float32
        u, v = r.uniform(-1, 1, (nk, nj + 4, ni + 4)).astype(npd), r.uniform(-1, 1, (nk, nj, ni)).astype(npd)
        out, total = (fields.alloc(ni, nj, nk, dtype, "cuda", halo=0, fill=0.0) for _ in range(2))
        mirror(fields.from_padded(u, dtype, "cuda"), fields.from_interior(v, dtype, "cuda"), out, total, alpha=0.375,
               domain=(ni, nj, nk))
        torch.cuda.synchronize()
        for got, want in zip((out, total), _mirror(u, v, 0.375)):
            assert np.array_equal(fields.interior(got, ni, nj, nk).cpu().numpy(), want)


@pytest.mark.gpu
@pytest.mark.parametrize("dims", [(1, 1, 1), (65, 7, 2), (130, 4, 9)], ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("dtype", DTYPES, ids=IDS)
def test_pair(dtype, dims):
    ni, nj, nk = dims
    print(f"pair {dims} {dtype}", flush=True)
    r = np.random.default_rng(1100 + nk)
    npd = np.float64 if dtype == torch.float64 else np.float32
    u, v = (r.uniform(-1, 1, (nk, nj + 4, ni + 4)).astype(npd) for _ in range(2))
    out = fields.alloc(ni, nj, nk, dtype, "cuda", halo=0, fill=0.0)
    pair(fields.from_padded(u, dtype, "cuda"), fields.from_padded(v, dtype, "cuda"), out, domain=dims)
    torch.cuda.synchronize()
    want = u[:, 2:-2, 2:-2].copy()
    want[:-1] = (u[1:, 2:-2, 3:-1] - u[:-1, 2:-2, 1:-3]) * v[:-1, 4:, 2:-2] + v[:-1, 2:-2, 2:-2]
    assert np.array_equal(fields.interior(out, ni, nj, nk).cpu().numpy(), want)
    rough(fields.from_padded(u, dtype, "cuda"), out, domain=dims)
    torch.cuda.synchronize()
    t = np.sqrt(u * u + npd(1))
    assert np.array_equal(fields.interior(out, ni, nj, nk).cpu().numpy(), t[:, 2:-2, 3:-1] - t[:, 1:-3, 2:-2])
