"""1D FP64 solves of 1 to 15 points in one launch against the oracle: cycle
counts, histories and solutions, zero starts and the cycle limit."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1210_7774_amd as M
from paper_1210_7774_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 7, 15])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 3), (0, 1)])
@pytest.mark.parametrize("zero", [False, True])
def test_solve_matches_oracle(n, nu1, nu2, zero):
    print("small 1D solve", n, nu1, nu2, zero, flush=True)
    f = I.normal_rhs(n, 1, 131)
    u0 = np.zeros(n) if zero else 1e-2 * I.normal_rhs(n, 1, 132)
    for rtol, maxc in ((1e-10, 100), (1e-10, 1), (1.0, 100)):
        want = u0.copy()
        hist = [np.linalg.norm(O.residual(want, f)) / np.linalg.norm(f)]
        while hist[-1] > rtol and len(hist) <= maxc:
            O.vcycle(want, f, opts=O.Opts(nu1=nu1, nu2=nu2, ncoarse=1))
            hist.append(np.linalg.norm(O.residual(want, f)) / np.linalg.norm(f))
        s = M.Solver(n, 1, nu1=nu1, nu2=nu2, max_cycles=maxc, zero_start=zero)
        u = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") if zero else torch.from_numpy(u0.copy()).to("cuda")
        rc, st = s.solve(u, torch.from_numpy(f).to("cuda"), rtol=rtol, raise_on_error=False)
        s.close()
        assert st.cycles == len(hist) - 1
        assert rc == (0 if hist[-1] <= rtol else M._abi.MG_NOT_CONVERGED)
        # residuals near the rounding floor (eps |A| |u| <= eps 4 (n + 1)^2 |f| / 8) agree to it
        assert np.allclose(st.history(), hist, rtol=1e-9, atol=1e-15 * (n + 1) ** 2)
        assert np.abs(u.cpu().numpy() - want).max() <= 1e-12 * max(np.abs(want).max(), np.abs(f).max())
