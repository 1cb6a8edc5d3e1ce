"""The training kernels at the sizes where their tiling can go wrong: rows of
less than, exactly and more than one 16-pixel tile, row counts that leave
remainders of the four-row (convolution) and eight-row (weight gradient) runs,
the smallest patch, and a batch with more runs than one launch of weight-
gradient blocks (each block then takes several)."""
import numpy as np
import pytest
import torch

import oracle.learned as LN
from paper_1210_7774_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("B,P,border", [(1, 3, 0), (2, 7, 0), (3, 16, 5), (2, 17, 5), (1, 31, 5), (5, 33, 3),
                                        (150, 33, 5)])
def test_gradient_at_tile_remainders(B, P, border):
    import paper_1210_7774_amd.learned as L
    print("learned gradient", B, P, border, flush=True)
    rng = np.random.default_rng(1000 * P + B)
    s = rng.standard_normal((B, P, P)).astype(np.float32)
    e = rng.standard_normal((B, P, P)).astype(np.float32)
    a = np.exp(rng.standard_normal((B, P, P))).astype(np.float32)
    w = I.he_normal_weights(21)
    loss, grad = L.loss_grad(dev(s), dev(e), dev(a), dev(w), border=border)
    want_loss, want = LN.loss_and_grad(s.astype(np.float64), e.astype(np.float64), a.astype(np.float64),
                                   w.astype(np.float64), border=border, bf16_emul=True)
    got = grad.cpu().numpy().astype(np.float64)
    # the bounds of the other gradient tests: FP32 sums, gradient signals
    # between layers stored in bfloat16 (2^-9 relative each)
    assert abs(loss - want_loss) <= 1e-4 * abs(want_loss)
    assert np.linalg.norm(got - want) <= 2e-2 * np.linalg.norm(want)
    # layers 1 and 4 by themselves (their products share no code path with 2 and 3)
    for sl in (slice(0, 144), slice(4896 - 144, 4896)):
        assert np.linalg.norm(got[sl] - want[sl]) <= 3e-2 * np.linalg.norm(want[sl])
