"""The register-resident 2D tail against the oracle: every top level it runs
(7, 15, 31 and 63 points, alone and below a tiled level), a non-zero starting
state on the tail's own top level, sweep counts that differ, every state type
and both operators, and several systems in one launch.  Bounds as in the other
cycle tests: 1e-12 (FP64 cycles), 2e-5 (FP32 refinement step), 3e-2 (bfloat16
state)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1210_7774_amd as M
from paper_1210_7774_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def rel(x, y):
    return float(np.abs(x - y).max() / np.abs(y).max())


@pytest.mark.parametrize("n", [7, 15, 31, 63, 127])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 3), (0, 1)])
@pytest.mark.parametrize("prec,vc", [("f64", False), ("f64", True), ("f32", False), ("f32", True), ("bf16", True)])
def test_tail_matches_oracle(n, nu1, nu2, prec, vc):
    print("tail2d", n, nu1, nu2, prec, vc, flush=True)
    a = I.lognormal_coef_2d(n, 4080) if vc else None
    f, u0 = I.normal_rhs(n, 2, 71), 1e-3 * I.normal_rhs(n, 2, 72)
    opts = O.Opts(nu1=nu1, nu2=nu2)
    s = M.Solver(n, 2, a=dev(a) if vc else None, nu1=nu1, nu2=nu2, precision=prec)
    u = dev(u0)
    s.vcycle(u, dev(f))
    if prec == "f64":
        want = u0.copy()
        O.vcycle(want, f, a=a, opts=opts)
        assert rel(u.cpu().numpy(), want) <= 1e-12
    else:
        ref = O.solve_ir(f, a=a, prec=O.F32 if prec == "f32" else O.BF16, tol=0.0, maxc=1, opts=opts, u0=u0)
        assert rel(u.cpu().numpy(), ref.u) <= (2e-5 if prec == "f32" else 3e-2)
    s.close()


def test_tail_of_a_batch():
    """One workgroup per system: each system's result is its own solve's."""
    ns = [127, 255, 127]
    coefs = [dev(I.lognormal_coef_2d(n, 4090 + k)) for k, n in enumerate(ns)]
    fs = [dev(I.normal_rhs(n, 2, 75 + k)) for k, n in enumerate(ns)]
    us = [torch.zeros(n, n, dtype=torch.float64, device="cuda") for n in ns]
    bs = M.BatchSolver(ns, coefs=coefs, precision="f32")
    rc, _ = bs.solve(us, fs, rtol=1e-10)
    assert rc == 0
    for n, a, f, u in zip(ns, coefs, fs, us):
        r = O.residual(u.cpu().numpy(), f.cpu().numpy(), a=a.cpu().numpy())
        assert np.linalg.norm(r) <= 1e-10 * float(f.norm())
    bs.close()
