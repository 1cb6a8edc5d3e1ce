"""Solves on arrays with padded rows and planes: the points end as the
contiguous solve's, and what lies between the rows keeps its contents."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1210_7774_amd import _abi
from paper_1210_7774_amd import inputs as I

pytestmark = pytest.mark.gpu
FILL = 7.5


def padded(n, dim, row, plane):
    """An array of FILL with row pitch `row` (and `plane` rows a plane), and a
    view of its n^dim points."""
    t = torch.full((n, row) if dim == 2 else (n, plane, row), FILL, dtype=torch.float64, device="cuda")
    return t, t[:, :n] if dim == 2 else t[:, :n, :n]


def solve(n, dim, u, f, row, plane, rtol, a=None, **opts):
    L = _abi.lib()
    g, o, st = _abi.Grid(), _abi.Options(), _abi.Stats()
    op = _abi.Operator(_abi.MG_OP_DIFFUSION if a is not None else _abi.MG_OP_POISSON,
                       ctypes.c_void_p(a.data_ptr()) if a is not None else None)
    L.mg_options_default(ctypes.byref(o))
    g.dim = dim
    for ax in range(3):
        g.n[ax], g.pitch[ax] = n if ax < dim else 1, 0
    g.pitch[1] = row
    if dim == 3:
        g.pitch[2] = row * plane
    for k, v in opts.items():
        setattr(o, k, v)
    nbytes, h = ctypes.c_size_t(0), ctypes.c_void_p(0)
    assert L.mg_workspace_size(ctypes.byref(g), ctypes.byref(op), ctypes.byref(o), ctypes.byref(nbytes)) == 0
    ws = torch.empty(nbytes.value, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    assert L.mg_setup(ctypes.byref(g), ctypes.byref(op), ctypes.byref(o), ctypes.c_void_p(ws.data_ptr()), nbytes,
                      ctypes.byref(h)) == 0
    rc = L.mg_solve(h, ctypes.c_void_p(u.data_ptr()), ctypes.c_void_p(f.data_ptr()), rtol, ctypes.byref(st))
    L.mg_destroy(h)
    return rc, st.cycles


JAC, F32 = dict(smoother=_abi.MG_SM_JACOBI), dict(precision=_abi.MG_P_F32_IR)


@pytest.mark.parametrize("dim,n,row,plane,opts", [
    (2, 63, 65, 0, {}), (2, 127, 130, 0, {}), (2, 255, 256, 0, {}), (2, 255, 260, 0, dict(nu1=3, nu2=3)),
    (2, 255, 301, 0, dict(cycle=_abi.MG_CYCLE_W)), (2, 255, 260, 0, dict(fmg=1)), (2, 255, 257, 0, F32),
    (2, 255, 260, 0, dict(use_graph=1)), (2, 2047, 2050, 0, {}), (2, 127, 140, 0, JAC), (2, 127, 129, 0, dict(nu2=1)),
    (3, 31, 34, 33, {}), (3, 31, 34, 31, JAC), (3, 31, 31, 35, dict(nu2=1)), (3, 31, 34, 33, F32)])
@pytest.mark.parametrize("vc", [False, True])
def test_padded_solve(dim, n, row, plane, opts, vc):
    if vc and dim == 3:
        pytest.skip("no diffusion operator in 3D")
    print("padded solve", dim, n, row, plane, opts, vc, flush=True)
    f = torch.from_numpy(np.ascontiguousarray(I.normal_rhs(n, dim, 55))).to("cuda")
    a = torch.from_numpy(np.ascontiguousarray(I.lognormal_coef_2d(n, 56))).to("cuda") if vc else None
    uc = torch.zeros_like(f)
    want = solve(n, dim, uc, f, n, n, 1e-8, a, **opts)
    (ut, uv), (ft, fv) = padded(n, dim, row, plane), padded(n, dim, row, plane)
    uv.zero_()
    fv.copy_(f)
    got = solve(n, dim, ut, ft, row, plane, 1e-8, a, **opts)
    assert got == want
    assert torch.equal(uv, uc)
    uv.fill_(FILL)
    assert bool((ut == FILL).all())


@pytest.mark.parametrize("dim,n,row,plane,fmg", [(3, 31, 34, 31, 0), (3, 31, 31, 33, 0), (3, 63, 70, 64, 0),
                                                 (3, 31, 34, 33, 1), (2, 63, 65, 0, 1), (2, 255, 260, 0, 1)])
def test_padded_zero_start(dim, n, row, plane, fmg):
    """u is not read; a solve that its first norm ends (a tolerance of 1, f = 0)
    leaves u = 0."""
    print("padded zero start", dim, n, row, plane, fmg, flush=True)
    fn = torch.from_numpy(np.ascontiguousarray(I.normal_rhs(n, dim, 55))).to("cuda")
    for rtol, rhs in ((1e-9, fn), (1.0, fn), (1e-9, torch.zeros_like(fn))):
        uc = torch.full_like(fn, FILL)
        want = solve(n, dim, uc, rhs, n, n, rtol, zero_start=1, fmg=fmg)
        (ut, uv), (ft, fv) = padded(n, dim, row, plane), padded(n, dim, row, plane)
        fv.copy_(rhs)
        got = solve(n, dim, ut, ft, row, plane, rtol, zero_start=1, fmg=fmg)
        assert got == want
        assert torch.equal(uv, uc)
        if want[1] == 0:
            assert float(uv.abs().max()) == 0.0
        uv.fill_(FILL)
        assert bool((ut == FILL).all())
