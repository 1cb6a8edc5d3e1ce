"""What a tune entry says is what runs: the launches of a solve, by their
timing classes ("pre n=" marches, "pre_tile n=" runs tiles), against the
entries a caller sets, the tuner reports and a cache file restores."""
import numpy as np
import pytest
import torch

import paper_1210_7774_amd as M
from paper_1210_7774_amd import inputs as I

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def run(s, n, f):
    """The solution, and which of "march" / "tile" the level of n points ran."""
    u = torch.zeros_like(f)
    s.profile(True)
    rc, _ = s.solve(u, f, rtol=1e-9)
    assert rc == 0
    names = set(s.kernel_timings())
    s.profile(False)
    forms = {form for form, name in (("march", "pre n=%d" % n), ("tile", "pre_tile n=%d" % n)) if name in names}
    assert len(forms) == 1
    return u, forms.pop()


@pytest.mark.parametrize("n,entry,want", [(255, None, "tile"), (255, (64, False), "march"), (255, (6, False), "march"),
                                          (255, (4, True), "tile"), (255, (8, None), "tile"),
                                          (1023, (32, False), "march"), (2047, (32, True), "march"),
                                          (2047, (32, None), "march")])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_entry_of_a_finest_size(n, entry, want, prec):
    print("tune entry", n, entry, prec, flush=True)
    f = dev(I.normal_rhs(n, 2, 141))
    s = M.Solver(n, 2, precision=prec)
    ref, _ = run(s, n, f)
    if entry:
        s.tune_set({n: entry})
        assert s.tune_get() == {n: entry}
    u, form = run(s, n, f)
    assert form == want
    assert float((u - ref).abs().max()) <= (1e-10 if prec == "f64" else 1e-6) * float(ref.abs().max())
    s.close()


@pytest.mark.parametrize("n,prec", [(255, "f64"), (511, "f32"), (1023, "f64")])
def test_tuner_reports_what_runs(n, prec, tmp_path):
    print("tuner", n, prec, flush=True)
    f = dev(I.normal_rhs(n, 2, 142))
    path = str(tmp_path / "tune.json")
    out = []
    for _ in range(2):  # (the second from the file)
        s = M.Solver(n, 2, precision=prec)
        choice = s.autotune(torch.zeros_like(f), f, reps=3, cache=path)
        u, form = run(s, n, f)
        out.append((choice, form, u))
        s.close()
    (c0, f0, u0), (c1, f1, u1) = out
    assert c0 == c1 and f0 == f1 and torch.equal(u0, u1)
    assert f0 == ("march" if c0[n][1] is False else "tile")
    assert c0[n][1] is False or c0[n][0] in (16, 32)
