"""A NaN or an infinity in one system of a batch: it goes through the pivot and
norm searches of every phase (maxima over lanes and waves), leaves no trace in
the systems beside it, which keep the factor they have alone bit for bit, and
its own system is reported as not solved."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2101_01763_amd as sp  # noqa: E402
from synth.dg_euler import DGConfig, make_problem  # noqa: E402


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("n,p,L,level", [(8, 1, 3, "leaf"), (8, 1, 3, "separator"), (12, 2, 4, "separator")])
def test_batch_with_one_bad_system(n, p, L, level, bad, dtype):
    cfg = DGConfig(n=n, p=p, seed=3)
    A, _, b, _ = make_problem(cfg)
    node = sp.nd(n, n, True, False, L)["node_of_elem"]
    e = int(np.argmax(node) if level == "leaf" else np.argmin(node))
    t = int(A.rowptr[e] + np.nonzero(A.colind[A.rowptr[e]:A.rowptr[e + 1]] == e)[0][0])
    val = A.val.copy()
    val[t, 1, 2] = bad
    good, poor = (sp.BSRMatrix.from_numpy(A.rowptr, A.colind, v) for v in (A.val, val))
    Fs = sp.factor_batched([(m, n, n, True, False) for m in (good, poor, good)], eps=1e-2, nlevels=L, dtype=dtype)
    one = sp.factor(good, n, n, True, False, eps=1e-2, nlevels=L, dtype=dtype)
    r = torch.as_tensor(b, device="cuda")
    x, xt = one.apply(r), one.apply_T(r)
    assert torch.isfinite(x).all() and torch.isfinite(xt).all()
    for F in (Fs[0], Fs[2]):
        assert F.stats()["size_after"] == one.stats()["size_after"]
        assert torch.equal(F.apply(r), x) and torch.equal(F.apply_T(r), xt)
    _, info = sp.solve(poor, r, Fs[1], s=4, restart=40, rtol=1e-8, maxit=40)
    assert not info.converged
