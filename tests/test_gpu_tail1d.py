"""1D cycles and solves in one wavefront against the oracle: every size they
run (31 .. 2047: one to 32 points a lane) and the first one they do not, sweep
counts that differ, a non-zero start, every state type; the one-launch solve's
history, cycle limit, restart across launches and error paths, and its
agreement with the launch-per-operation form (captured cycles)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1210_7774_amd as M
from paper_1210_7774_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("n", [31, 63, 127, 255, 1023, 2047, 4095])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (1, 3), (0, 1)])
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
def test_cycle_matches_oracle(n, nu1, nu2, prec):
    print("tail1d", n, nu1, nu2, prec, flush=True)
    f, u0 = I.sine_plus_noise_1d(n, 121), 1e-2 * I.normal_rhs(n, 1, 122)
    opts = O.Opts(nu1=nu1, nu2=nu2, ncoarse=1)
    s = M.Solver(n, 1, nu1=nu1, nu2=nu2, precision=prec)
    u = dev(u0)
    s.vcycle(u, dev(f))
    got = u.cpu().numpy()
    if prec == "f64":
        want = u0.copy()
        O.vcycle(want, f, opts=opts)
        assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()
    else:
        # (an FP32 step computes the correction in FP32: bounds of the correction)
        ref = O.solve_ir(f, prec=O.F32 if prec == "f32" else O.BF16, tol=0.0, maxc=1, opts=opts, u0=u0)
        assert np.abs(got - ref.u).max() <= (2e-5 if prec == "f32" else 3e-2) * np.abs(ref.u - u0).max()
    s.close()


@pytest.mark.parametrize("n", [31, 63, 511, 2047])
@pytest.mark.parametrize("nu1,nu2", [(2, 2), (0, 1)])
def test_solve_matches_captured_cycles(n, nu1, nu2):
    """nu 0 + 1 converges slowly: more cycles than one launch takes."""
    f = dev(I.normal_rhs(n, 1, 123))
    out = []
    for graph in (False, True):
        s = M.Solver(n, 1, nu1=nu1, nu2=nu2, use_graph=graph, max_cycles=150)
        u = dev(1e-3 * I.normal_rhs(n, 1, 124))
        rc, st = s.solve(u, f, rtol=1e-9, raise_on_error=False)
        out.append((rc, st.cycles, np.array(st.history()), u.cpu().numpy()))
        s.close()
    (rc0, c0, h0, u0), (rc1, c1, h1, u1) = out
    assert rc0 == rc1 and c0 == c1 and len(h0) == len(h1)
    assert np.abs(u0 - u1).max() <= 1e-12 * np.abs(u1).max()
    # norms near the rounding floor of the residual (eps |A| |u|) agree to it
    floor = 1e-16 * 4.0 * (n + 1) ** 2 * np.abs(u1).max() * np.sqrt(n) / float(f.norm())
    assert np.all(np.abs(h0 - h1) <= 1e-9 * h1 + 10 * floor)


def test_solve_limits():
    n = 255
    f = dev(I.sine_plus_noise_1d(n, 125))
    s = M.Solver(n, 1, nu1=0, nu2=1, max_cycles=2)
    u = torch.zeros(n, dtype=torch.float64, device="cuda")
    rc, st = s.solve(u, f, rtol=1e-13, raise_on_error=False)
    assert rc == M._abi.MG_NOT_CONVERGED and st.cycles == 2
    bad = f.clone()
    bad[7] = float("inf")
    rc, st = s.solve(u, bad, rtol=1e-9, raise_on_error=False)
    assert rc == M._abi.MG_ERR_NONFINITE and st.cycles == 0
    s.close()
