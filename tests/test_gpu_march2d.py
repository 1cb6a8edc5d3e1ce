"""The row-marching 2D kernels with every level above the tail marching
(MGX_TILE_MAX=0), against the oracle: block heights that give items wholly
inside the domain (their own branch-free form), items on each edge, and ragged
last strips and blocks; one and two column groups; every state type and both
operators.  Bounds as in the other cycle tests: 1e-12 of the iterate for FP64
cycles; a refinement step is what FP32 arithmetic computes, so its 2e-5 (3e-2
with a bfloat16-stored iterate) is of the largest correction."""
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


@pytest.mark.parametrize("n,nu,hb,g", [(127, 2, 4, 1), (511, 1, 10, 1), (511, 2, 30, 1), (511, 3, 64, 1),
                                       (511, 2, 16, 2), (511, 2, 256, 1)])
@pytest.mark.parametrize("prec,vc", [("f64", False), ("f64", True), ("f32", True), ("bf16", False)])
def test_marching_matches_oracle(n, nu, hb, g, prec, vc, monkeypatch):
    print("marching", n, nu, hb, g, prec, vc, flush=True)
    for k, v in (("TILE_MAX", 0), ("HB", hb), ("G", g)):
        monkeypatch.setenv("MGX_" + k, str(v))
    a = I.lognormal_coef_2d(n, 4095) if vc else None
    f, u0 = I.normal_rhs(n, 2, 101), 1e-3 * I.normal_rhs(n, 2, 102)
    opts = O.Opts(nu1=nu, nu2=nu)
    s = M.Solver(n, 2, a=dev(a) if vc else None, nu1=nu, nu2=nu, precision=prec)
    u = dev(u0)
    s.vcycle(u, dev(f))
    if prec == "f64":
        want = u0.copy()
        O.vcycle(want, f, a=a, opts=opts)
        assert rel(u.cpu().numpy(), want) <= 1e-12
    else:
        ref = O.solve_ir(f, a=a, prec=O.F32 if prec == "f32" else O.BF16, tol=0.0, maxc=1, opts=opts, u0=u0)
        err = np.abs(u.cpu().numpy() - ref.u).max()
        assert err <= (2e-5 if prec == "f32" else 3e-2) * np.abs(ref.u - u0).max()
    s.close()
