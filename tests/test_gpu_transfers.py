"""The 2D residual + restriction and prolongation + correction of the levels
that smooth point by point (weighted Jacobi here) against the oracle, at sizes
with ragged strips (30 coarse columns; 64 fine ones) and row runs, both
operators, each state type; and a learned cycle from a start
that is not read against one from a zeroed array."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1210_7774_amd as M
from paper_1210_7774_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("n", [127, 255, 1023])
@pytest.mark.parametrize("vc", [False, True])
def test_level_transfers(n, vc):
    print("transfers", n, vc, flush=True)
    a = I.lognormal_coef_2d(n, 4131) if vc else None
    s = M.Solver(n, 2, a=dev(a) if vc else None, smoother="jacobi", nu1=1, nu2=1)
    u0, f = I.normal_rhs(n, 2, 131), I.normal_rhs(n, 2, 132)
    nc = (n - 1) // 2
    uc = I.normal_rhs(nc, 2, 133)
    uo = torch.empty(n, n, dtype=torch.float64, device="cuda")
    fc = torch.empty(nc, nc, dtype=torch.float64, device="cuda")
    s.smooth_restrict(dev(u0), dev(f), uo, fc)
    want = O.sweep(u0.copy(), f, a=a, kind=O.JACOBI, nsweeps=1)
    wfc = O.restrict(O.residual(want, f, a=a))
    assert np.abs(uo.cpu().numpy() - want).max() <= 1e-13 * np.abs(want).max()
    assert np.abs(fc.cpu().numpy() - wfc).max() <= 1e-13 * np.abs(wfc).max()
    s.correct_smooth(dev(u0), dev(uc), dev(f), uo)
    want = O.prolong_add(uc, u0.copy())
    O.sweep(want, f, a=a, kind=O.JACOBI, nsweeps=1)
    assert np.abs(uo.cpu().numpy() - want).max() <= 1e-13 * np.abs(want).max()
    s.close()


@pytest.mark.parametrize("n,vc,prec", [(127, False, "f64"), (511, True, "f64"), (255, True, "f32"),
                                       (511, False, "f32"), (255, True, "bf16")])
def test_jacobi_cycle(n, vc, prec):
    print("jacobi cycle", n, vc, prec, flush=True)
    a = I.lognormal_coef_2d(n, 4132) if vc else None
    f, u0 = I.normal_rhs(n, 2, 134), 1e-5 * I.normal_rhs(n, 2, 135)
    s = M.Solver(n, 2, a=dev(a) if vc else None, smoother="jacobi", precision=prec)
    opts = O.Opts(smoother=O.JACOBI)
    if prec == "f64":
        u, fd = dev(u0), dev(f)
        s.vcycle(u, fd)
        want = u0.copy()
        O.vcycle(want, f, a=a, opts=opts)
        assert np.abs(u.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
    else:
        u = dev(u0)
        s.vcycle(u, dev(f))
        ref = O.solve_ir(f, a=a, prec=O.F32 if prec == "f32" else O.BF16, tol=0.0, maxc=1, opts=opts, u0=u0)
        # (the step computes the correction in its own precision)
        bound = (2e-5 if prec == "f32" else 3e-2) * np.abs(ref.u - u0).max()
        assert np.abs(u.cpu().numpy() - ref.u).max() <= bound
    s.close()


@pytest.mark.parametrize("n,prec", [(127, "f32"), (255, "bf16"), (255, "f32")])
def test_learned_cycles_repeat(n, prec):
    """Each cycle's first learned step starts from 0 without reading its
    array: solves that follow each other on one handle (the array then holds
    the last correction) agree bit for bit with a fresh handle's."""
    import paper_1210_7774_amd.learned as L
    a, f = I.lognormal_coef_2d(n, 4133), dev(I.normal_rhs(n, 2, 136))
    out = []
    for fresh in (True, False):
        s = M.Solver(n, 2, a=dev(a), smoother="learned", precision=prec, learned=L.jacobi_start(), max_cycles=3)
        if not fresh:
            w = torch.zeros(n, n, dtype=torch.float64, device="cuda")
            s.solve(w, dev(I.normal_rhs(n, 2, 137)), rtol=1e-30, raise_on_error=False)
        u = torch.zeros(n, n, dtype=torch.float64, device="cuda")
        s.solve(u, f, rtol=1e-30, raise_on_error=False)
        out.append(u.cpu().numpy())
        s.close()
    assert np.array_equal(out[0], out[1])
