"""Solves whose first norm already ends them, and zero starts of every path: u
is never read and ends as the zeroed-u solve's, also when no cycle runs (f = 0,
whose relative residual is not a number, and a tolerance of 1); one-cycle
limits; a captured cycle."""
import numpy as np
import pytest
import torch

import paper_1210_7774_amd as M
from paper_1210_7774_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


CASES = [(1, 255, "f64", {}), (2, 63, "f64", {}), (2, 255, "f64", {}), (2, 255, "f64", {"cycle": "W"}),
         (2, 255, "f64", {"smoother": "jacobi"}), (2, 255, "f32", {}), (2, 255, "f64", {"fmg": True}),
         (2, 255, "f64", {"use_graph": True}), (3, 31, "f64", {}), (3, 31, "bf16", {})]


@pytest.mark.parametrize("dim,n,prec,opt", CASES)
def test_zero_start_equals_zeroed_u(dim, n, prec, opt):
    print("zero start", dim, n, prec, opt, flush=True)
    f = dev(I.normal_rhs(n, dim, 111))
    for rtol, maxc in ((1e-9, 100), (1e-9, 1), (1e-9, 3), (1.0, 100)):
        out = []
        for zs in (False, True):
            s = M.Solver(n, dim, precision=prec, zero_start=zs, max_cycles=maxc, **opt)
            u = torch.zeros((n,) * dim, dtype=torch.float64, device="cuda")
            for _ in range(2):  # (a second solve on the handle too)
                u.fill_(float("nan") if zs else 0.0)
                rc, st = s.solve(u, f, rtol=rtol, raise_on_error=False)
            out.append((rc, st.cycles, st.history(), u.cpu().numpy()))
            s.close()
        assert out[0][:2] == out[1][:2]
        assert np.array_equal(out[0][2], out[1][2]) and np.array_equal(out[0][3], out[1][3])


@pytest.mark.parametrize("dim,n,prec,opt", CASES)
def test_zero_rhs(dim, n, prec, opt):
    """f = 0: the relative residual is 0 / 0, a non-finite norm; u ends as the
    zero it started from."""
    f = torch.zeros((n,) * dim, dtype=torch.float64, device="cuda")
    s = M.Solver(n, dim, precision=prec, zero_start=True, **opt)
    u = torch.full_like(f, 3.0)
    rc, st = s.solve(u, f, rtol=1e-9, raise_on_error=False)
    assert rc == M._abi.MG_ERR_NONFINITE and st.cycles == 0
    assert float(u.abs().max()) == 0.0
    s.close()
