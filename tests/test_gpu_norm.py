"""The FP64 residual norm and residual against the oracle at the sizes where
the 2D strips (64 columns) and row runs (8 rows) leave remainders, below one
strip, and in 1D and 3D (runs of 8 and 32 planes), both operators, single
systems and batches.  The residual itself is a sum of five or seven terms
(1e-13 of the largest), the norm adds n^d of its squares (1e-12)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_1210_7774_amd as M
from paper_1210_7774_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("dim,n,vc", [(1, 63, False), (2, 3, True), (2, 7, True), (2, 63, True), (2, 127, True),
                                      (2, 255, False), (2, 1023, True), (3, 7, False), (3, 127, False)])
def test_residual_and_norm(dim, n, vc):
    print("norm", dim, n, vc, flush=True)
    a = I.lognormal_coef_2d(n, 4085) if vc else None
    f, u = I.normal_rhs(n, dim, 91), 1e-2 * I.normal_rhs(n, dim, 92)
    s = M.Solver(n, dim, a=dev(a) if vc else None)
    r = torch.empty((n,) * dim, dtype=torch.float64, device="cuda")
    s.residual(dev(u), dev(f), r)
    want = O.residual(u, f, a=a)
    assert np.abs(r.cpu().numpy() - want).max() <= 1e-13 * np.abs(want).max()
    rel = s.residual_norm(dev(u), dev(f))
    assert abs(rel / (np.linalg.norm(want) / np.linalg.norm(f)) - 1.0) <= 1e-12
    s.close()


def test_batched_first_norm():
    """A batch's initial residual norms (max_cycles 1: hist[0] is the norm of
    the initial guess)."""
    ns = [127, 255, 1023]
    coefs = [I.lognormal_coef_2d(n, 4086 + k) for k, n in enumerate(ns)]
    fs, us = [I.normal_rhs(n, 2, 93) for n in ns], [1e-2 * I.normal_rhs(n, 2, 94) for n in ns]
    bs = M.BatchSolver(ns, coefs=[dev(a) for a in coefs], precision="f32", max_cycles=1)
    _, stats = bs.solve([dev(u) for u in us], [dev(f) for f in fs], rtol=1e-30, raise_on_error=False)
    for a, f, u, st in zip(coefs, fs, us, stats):
        want = np.linalg.norm(O.residual(u, f, a=a)) / np.linalg.norm(f)
        assert abs(st.hist[0] / want - 1.0) <= 1e-12
    bs.close()
