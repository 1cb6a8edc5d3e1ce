"""The LDS-tiled 2D level kernels on every level above the tail, the finest
included, against the oracle: sizes that take each tile edge (16 where 32
leaves CUs idle, 32, and 28 for three sweeps) with a ragged last tile, the
smallest level above the tail, every state type, and both operators.  The
bounds are those of the other cycle tests: 1e-12 of the iterate for FP64
cycles, 2e-5 for a refinement step with FP32 cycles, 3e-2 with a bfloat16-
stored iterate, 1e-6 for residual norms."""
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


@pytest.mark.parametrize("n,nu", [(127, 1), (127, 2), (127, 3), (511, 1), (511, 2), (511, 3)])
@pytest.mark.parametrize("prec,vc", [("f64", False), ("f64", True), ("f32", False), ("f32", True), ("bf16", True)])
def test_tiled_finest_matches_oracle(n, nu, prec, vc):
    print("tiled finest", n, nu, prec, vc, flush=True)
    a = I.lognormal_coef_2d(n, 4060) if vc else None
    f = I.normal_rhs(n, 2, 61)
    opts = O.Opts(nu1=nu, nu2=nu)
    s = M.Solver(n, 2, a=dev(a) if vc else None, nu1=nu, nu2=nu, precision=prec, max_cycles=2)
    u, v = (torch.zeros(n, n, dtype=torch.float64, device="cuda") for _ in range(2))
    if prec == "f64":
        rc, st = s.solve(v, dev(f), rtol=1e-14, raise_on_error=False)
        want = np.zeros_like(f)
        for k in range(2):
            s.vcycle(u, dev(f))
            O.vcycle(want, f, a=a, opts=opts)
            assert rel(u.cpu().numpy(), want) <= 1e-12
            r = np.linalg.norm(O.residual(want, f, a=a)) / np.linalg.norm(f)
            assert abs(st.history()[k + 1] / r - 1.0) <= 1e-6
        assert rel(v.cpu().numpy(), want) <= 1e-12
    else:
        s.vcycle(u, dev(f))
        ref = O.solve_ir(f, a=a, prec=O.F32 if prec == "f32" else O.BF16, tol=0.0, maxc=1, opts=opts)
        assert rel(u.cpu().numpy(), ref.u) <= (2e-5 if prec == "f32" else 3e-2)
    s.close()
