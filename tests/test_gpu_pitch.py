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


def handle(n, row, opts):
    L = _abi.lib()
    g, o, op = _abi.Grid(), _abi.Options(), _abi.Operator(_abi.MG_OP_POISSON, None)
    L.mg_options_default(ctypes.byref(o))
    g.dim, g.n[0], g.n[1], g.n[2], g.pitch[1] = 2, n, n, 1, row
    for k, v in opts.items():
        setattr(o, k, v)
    nbytes, h = ctypes.c_size_t(0), ctypes.c_void_p(0)
    assert L.mg_workspace_size(ctypes.byref(g), ctypes.byref(op), ctypes.byref(o), ctypes.byref(nbytes)) == 0
    ws = torch.empty(nbytes.value, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    assert L.mg_setup(ctypes.byref(g), ctypes.byref(op), ctypes.byref(o), ctypes.c_void_p(ws.data_ptr()), nbytes,
                      ctypes.byref(h)) == 0
    return h, ws


@pytest.mark.parametrize("n,row,opts", [(255, 260, {}), (2047, 2049, {}), (127, 130, JAC)])
def test_padded_level_operations(n, row, opts):
    print("padded level operations", n, row, opts, flush=True)
    L, nc = _abi.lib(), (n - 1) // 2
    u, f, uc = (torch.from_numpy(np.ascontiguousarray(I.normal_rhs(m, 2, 60 + m % 7))).to("cuda") for m in (n, n, nc))
    f = f.flip(0).contiguous()
    outs = []
    for p in (n, row):
        h, ws = handle(n, p, opts)
        (ut, uv), (ft, fv), (ot, ov), (qt, qv) = (padded(n, 2, p, 0) for _ in range(4))
        uv.copy_(u)
        fv.copy_(f)
        fc, r, s = torch.empty_like(uc), torch.empty_like(u), torch.empty_like(u)
        ptr = [ctypes.c_void_p(t.data_ptr()) for t in (ut, ft, ot, fc, uc, qt, r, s)]
        assert L.mg_smooth_restrict(h, ptr[0], ptr[1], ptr[2], ptr[3]) == 0
        assert L.mg_correct_smooth(h, ptr[0], ptr[4], ptr[1], ptr[5]) == 0
        assert L.mg_residual(h, ptr[0], ptr[1], ptr[6]) == 0
        assert L.mg_scaled_residual(h, ptr[0], ptr[1], ptr[7]) == 0
        L.mg_destroy(h)
        outs.append([t.clone() for t in (ov, fc, qv, r, s)])
        for t, v in ((ot, ov), (qt, qv)):
            v.fill_(FILL)
            assert bool((t == FILL).all())
    for x, y in zip(*outs):
        assert torch.equal(x, y)


@pytest.mark.parametrize("prec", [_abi.MG_P_F64, _abi.MG_P_F32_IR])
def test_padded_batch(prec):
    print("padded batch", prec, flush=True)
    L, ns, rows = _abi.lib(), [127, 255, 511], [130, 255, 600]
    fs = [torch.from_numpy(np.ascontiguousarray(I.normal_rhs(n, 2, 66 + n))).to("cuda") for n in ns]
    outs = []
    for pitches in (ns, rows):
        g, ops, o = (_abi.Grid * 3)(), (_abi.Operator * 3)(), _abi.Options()
        L.mg_options_default(ctypes.byref(o))
        o.precision = prec
        us, ft = [], []
        for k, (n, p) in enumerate(zip(ns, pitches)):
            g[k].dim, g[k].n[0], g[k].n[1], g[k].n[2], g[k].pitch[1] = 2, n, n, 1, p
            ops[k] = _abi.Operator(_abi.MG_OP_POISSON, None)
            us.append(padded(n, 2, p, 0))
            us[-1][1].zero_()
            ft.append(padded(n, 2, p, 0))
            ft[-1][1].copy_(fs[k])
        nbytes, h = ctypes.c_size_t(0), ctypes.c_void_p(0)
        assert L.mg_workspace_size_batch(3, g, ops, ctypes.byref(o), ctypes.byref(nbytes)) == 0
        ws = torch.empty(nbytes.value, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        assert L.mg_setup_batch(3, g, ops, ctypes.byref(o), ctypes.c_void_p(ws.data_ptr()), nbytes, ctypes.byref(h)) == 0
        st = (_abi.Stats * 3)()
        up = (ctypes.c_void_p * 3)(*[t.data_ptr() for t, _ in us])
        fp = (ctypes.c_void_p * 3)(*[t.data_ptr() for t, _ in ft])
        assert L.mg_solve_batch(h, up, fp, 1e-8, st) == 0
        L.mg_destroy(h)
        outs.append(([s.cycles for s in st], [v.clone() for _, v in us]))
        for t, v in us:
            v.fill_(FILL)
            assert bool((t == FILL).all())
    assert outs[0][0] == outs[1][0]
    for x, y in zip(outs[0][1], outs[1][1]):
        assert torch.equal(x, y)
