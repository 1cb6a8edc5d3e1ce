"""1D full multigrid in one wavefront against the oracle: every size it runs
(31 .. 2047 points) and the first one it does not, each cycle type, sweep
counts that differ; the second of two passes overwrites the first's result
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


@pytest.mark.parametrize("n", [31, 63, 127, 1023, 2047, 4095])
@pytest.mark.parametrize("kind", ["V", "W", "F"])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 0)])
def test_fmg_pass_matches_oracle(n, kind, nu1, nu2):
    print("fmg 1d", n, kind, nu1, nu2, flush=True)
    s = M.Solver(n, 1, nu1=nu1, nu2=nu2, cycle=kind, fmg=True, max_cycles=1, ncoarse=1)
    f = I.sine_plus_noise_1d(n, 171)
    for k in range(2):
        u = dev(I.normal_rhs(n, 1, 172 + k))
        s.solve(u, dev(f), rtol=0.0, raise_on_error=False)
        want = O.fmg(f, opts=O.Opts(nu1=nu1, nu2=nu2, ncoarse=1), kind=kind)
        assert np.abs(u.cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
    s.close()
