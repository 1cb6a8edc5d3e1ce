"""W and F cycles, and full multigrid of them, with the coarse levels in the
register-resident 2D tail, against the oracle: every top level it runs (7 .. 63
points), alone and below tiled levels, both operators, sweep counts that
differ, every state type.  Bounds as in the other cycle tests: 1e-12 (FP64),
and of the largest correction 2e-5 (FP32 step) and 3e-2 (bfloat16 state)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1210_7774_amd as M
from paper_1210_7774_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("n", [7, 15, 31, 63, 127, 255])
@pytest.mark.parametrize("kind", ["W", "F"])
@pytest.mark.parametrize("vc", [False, True])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (0, 1), (1, 0)])
def test_cycle_matches_oracle(n, kind, vc, nu1, nu2):
    print("wf tail", n, kind, vc, nu1, nu2, flush=True)
    a = I.lognormal_coef_2d(n, 4151) if vc else None
    f, want = I.normal_rhs(n, 2, 151), 1e-3 * I.normal_rhs(n, 2, 152)
    s = M.Solver(n, 2, a=dev(a) if vc else None, nu1=nu1, nu2=nu2, cycle=kind)
    u = dev(want)
    for _ in range(2):
        s.vcycle(u, dev(f))
        O.cycle(want, f, a=a, opts=O.Opts(nu1=nu1, nu2=nu2), kind=kind)
        assert np.abs(u.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
    s.close()


@pytest.mark.parametrize("n,kind,vc", [(31, "W", True), (63, "F", False), (255, "F", True), (511, "W", False)])
def test_fmg_of_cycles(n, kind, vc):
    print("wf fmg", n, kind, vc, flush=True)
    a = I.lognormal_coef_2d(n, 4152) if vc else None
    f = I.normal_rhs(n, 2, 153)
    s = M.Solver(n, 2, a=dev(a) if vc else None, cycle=kind, fmg=True, max_cycles=1)
    u = dev(I.normal_rhs(n, 2, 154))
    s.solve(u, dev(f), rtol=0.0, raise_on_error=False)
    want = O.fmg(f, a=a, kind=kind)
    assert np.abs(u.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
    s.close()


@pytest.mark.parametrize("n,kind,vc,prec", [(31, "F", False, "f32"), (63, "W", True, "f32"), (127, "F", True, "f32"),
                                            (63, "F", True, "bf16"), (15, "W", False, "bf16")])
def test_refinement_step(n, kind, vc, prec):
    print("wf refinement", n, kind, vc, prec, flush=True)
    a = I.lognormal_coef_2d(n, 4153) if vc else None
    f, u0 = I.normal_rhs(n, 2, 155), 1e-5 * I.normal_rhs(n, 2, 156)
    s = M.Solver(n, 2, a=dev(a) if vc else None, cycle=kind, precision=prec)
    u = dev(u0)
    s.vcycle(u, dev(f))
    ref = O.solve_ir(f, a=a, prec=O.F32 if prec == "f32" else O.BF16, tol=0.0, maxc=1, u0=u0, kind=kind)
    assert np.abs(u.cpu().numpy() - ref.u).max() <= (2e-5 if prec == "f32" else 3e-2) * np.abs(ref.u - u0).max()
    s.close()
