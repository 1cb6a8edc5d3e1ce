"""Full multigrid of V-cycles with the coarse levels in the register-resident
tail, against the oracle: every top level it runs (7 .. 63 points; both
operators), alone and below tiled and marching levels, sweep counts that
differ, and interpolation onto levels whose last strip or rows are ragged
(1e-12, the bound of the other cycle tests)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1210_7774_amd as M
from paper_1210_7774_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("n", [7, 15, 31, 63, 127, 511])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 3)])
@pytest.mark.parametrize("vc", [False, True])
def test_fmg_pass_matches_oracle(n, nu1, nu2, vc):
    print("fmg tail", n, nu1, nu2, vc, flush=True)
    a = I.lognormal_coef_2d(n, 4141) if vc else None
    s = M.Solver(n, 2, a=dev(a) if vc else None, nu1=nu1, nu2=nu2, fmg=True, max_cycles=1)
    f = I.normal_rhs(n, 2, 141)
    for k in range(2):  # (the second pass overwrites the first one's result)
        u = dev(I.normal_rhs(n, 2, 142 + k))
        s.solve(u, dev(f), rtol=0.0, raise_on_error=False)
        want = O.fmg(f, a=a, opts=O.Opts(nu1=nu1, nu2=nu2))
        assert np.abs(u.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
    s.close()
