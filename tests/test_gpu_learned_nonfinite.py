"""Gradients with an infinity at the edge of a patch: an entry is finite
exactly where its sum over the pixels of the patch (zeros around it) is, so
rows that end inside a 16-pixel tile and taps that reach past a border add
and drop nothing."""
import numpy as np
import pytest
import torch

import oracle.learned as LN
import paper_1210_7774_amd.learned as L

pytestmark = pytest.mark.gpu


def finite_entries(s, e, a, w, border):
    """Which entries of the gradient are finite; values outside the window
    take no part in the energies, masked gradients are 0."""
    y, acts, ws = LN.forward(s, w, bf16_emul=True, keep=True)
    P = s.shape[-1]
    inside = np.zeros((P, P), dtype=bool)
    inside[border:P - border, border:P - border] = True
    r = np.where(inside, e - y, 0.0)
    g = (LN.energy_operator(r, a, border) * (-2.0 / len(s)) / LN.energy(np.where(inside, e, 0.0), a, border)[:, None, None])[:, None]
    grads = [None] * 4
    for li in range(3, -1, -1):
        grads[li] = LN.conv3x3_wgrad(acts[li], g)
        g = np.where(acts[li] > 0, LN.conv3x3_dgrad(g, ws[li]), 0.0)
    return np.isfinite(LN.flatten(grads))


@pytest.mark.parametrize("P", [16, 30, 33])
@pytest.mark.parametrize("where", ["s right", "s corner", "e corner"])
def test_gradient_is_finite_where_its_sums_are(P, where):
    print("non-finite gradient", P, where, flush=True)
    rng = np.random.default_rng(77)
    s, e = rng.standard_normal((2, P, P)).astype(np.float32), rng.standard_normal((2, P, P)).astype(np.float32)
    a = np.exp(0.5 * rng.standard_normal((2, P, P))).astype(np.float32)
    w = L.jacobi_start()
    x, border = (s, 5) if where[0] == "s" else (e, 0)
    x[1, P // 2 if where == "s right" else P - 1, P - 1] = np.inf
    with np.errstate(invalid="ignore"):
        want = finite_entries(s.astype(np.float64), e.astype(np.float64), a.astype(np.float64),
                              w.cpu().numpy().astype(np.float64), border)
    dev = [torch.from_numpy(t).to("cuda") for t in (s, e, a)]
    _, grad = L.loss_grad(*dev, w, border=border)
    got = np.isfinite(grad.cpu().numpy())
    assert 0 < want.sum() < want.size
    assert np.array_equal(got, want)
