"""The register-resident 3D tail against the oracle: both top levels it runs
(7 and 15 points, alone and below wavefront levels), a non-zero starting state
on the tail's own top level, sweep counts that differ, every state type.
Bounds as in the other cycle tests: 1e-12 (FP64 cycles), 2e-5 (FP32 refinement
step), 3e-2 (bfloat16 state)."""
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


@pytest.mark.parametrize("n", [7, 15, 31])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 3), (0, 1)])
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
def test_tail_matches_oracle(n, nu1, nu2, prec):
    print("tail3d", n, nu1, nu2, prec, flush=True)
    f, u0 = I.normal_rhs(n, 3, 81), 1e-3 * I.normal_rhs(n, 3, 82)
    opts = O.Opts(nu1=nu1, nu2=nu2)
    s = M.Solver(n, 3, nu1=nu1, nu2=nu2, precision=prec)
    u = dev(u0)
    s.vcycle(u, dev(f))
    if prec == "f64":
        want = u0.copy()
        O.vcycle(want, f, opts=opts)
        assert rel(u.cpu().numpy(), want) <= 1e-12
    else:
        ref = O.solve_ir(f, prec=O.F32 if prec == "f32" else O.BF16, tol=0.0, maxc=1, opts=opts, u0=u0)
        assert rel(u.cpu().numpy(), ref.u) <= (2e-5 if prec == "f32" else 3e-2)
    s.close()
