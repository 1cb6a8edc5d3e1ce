"""W and F cycles with the coarse levels in the register-resident 1D and 3D
tails, against the oracle: every 1D size they run (31 .. 2047 points), the 3D
tops 7 and 15 alone and below fused levels, sweep counts that differ, every
state type.  Bounds as in the other cycle tests: 1e-12 (FP64), and of the
largest correction 2e-5 (FP32 step) and 3e-2 (bfloat16 state)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1210_7774_amd as M
from paper_1210_7774_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("d,n", [(1, 31), (1, 63), (1, 127), (1, 1023), (1, 2047), (3, 7), (3, 15), (3, 31), (3, 63)])
@pytest.mark.parametrize("kind", ["W", "F"])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (0, 1), (1, 0)])
def test_cycle_matches_oracle(d, n, kind, nu1, nu2):
    print("wf tail", d, n, kind, nu1, nu2, flush=True)
    nco = 1 if d == 1 else 3
    f, want = I.normal_rhs(n, d, 161), 1e-3 * I.normal_rhs(n, d, 162)
    s = M.Solver(n, d, nu1=nu1, nu2=nu2, cycle=kind, ncoarse=nco)
    u = dev(want)
    for _ in range(2):
        s.vcycle(u, dev(f))
        O.cycle(want, f, opts=O.Opts(nu1=nu1, nu2=nu2, ncoarse=nco), kind=kind)
        assert np.abs(u.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
    s.close()


@pytest.mark.parametrize("d,n,kind,prec", [(1, 255, "F", "f32"), (1, 2047, "W", "bf16"), (3, 15, "W", "f32"),
                                           (3, 31, "F", "f32"), (3, 15, "F", "bf16")])
def test_refinement_step(d, n, kind, prec):
    print("wf refinement", d, n, kind, prec, flush=True)
    nco = 1 if d == 1 else 3
    f, u0 = I.normal_rhs(n, d, 163), 1e-5 * I.normal_rhs(n, d, 164)
    s = M.Solver(n, d, cycle=kind, precision=prec, ncoarse=nco)
    u = dev(u0)
    s.vcycle(u, dev(f))
    ref = O.solve_ir(f, prec=O.F32 if prec == "f32" else O.BF16, tol=0.0, maxc=1, u0=u0, kind=kind,
                     opts=O.Opts(ncoarse=nco))
    assert np.abs(u.cpu().numpy() - ref.u).max() <= (2e-5 if prec == "f32" else 3e-2) * np.abs(ref.u - u0).max()
    s.close()
