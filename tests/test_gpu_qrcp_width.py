"""Rank-revealing QR launches of up to 256 interfaces of more than 128 rows take
512 threads, larger ones 256: both sum in the same order, so a system factored
alone (fewer interfaces per launch) and in a batch must give the same ranks and
the same factor bit for bit, and eps = 0.1 .. 1e-3 walk through the block
widths' remainders."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2101_01763_amd as sp  # noqa: E402
from synth.dg_euler import DGConfig, make_problem  # noqa: E402


@pytest.mark.parametrize("n,p,L,nsys,dtype,eps", [
    (24, 3, 6, 8, "f32", 1e-2),    # 64 unknowns an element: 192 and 384 rows
    (24, 3, 6, 8, "f64", 1e-3),
    (33, 2, 7, 6, "f32", 1e-1),    # odd counts
    (33, 2, 6, 12, "f64", 1e-2),
])
def test_alone_and_in_a_batch(n, p, L, nsys, dtype, eps):
    cfg = DGConfig(n=n, p=p, seed=n)
    A, _, _, _ = make_problem(cfg)
    mat = sp.BSRMatrix.from_numpy(A.rowptr, A.colind, A.val)
    Fs = sp.factor_batched([(mat, n, n, True, False)] * nsys, eps=eps, nlevels=L, dtype=dtype)
    one = sp.factor(mat, n, n, True, False, eps=eps, nlevels=L, dtype=dtype)
    r = torch.as_tensor(np.random.default_rng(n).standard_normal(cfg.N), device="cuda")
    x, xt = one.apply(r), one.apply_T(r)
    for F in Fs:
        assert F.stats()["size_after"] == one.stats()["size_after"]
        assert torch.equal(F.apply(r), x) and torch.equal(F.apply_T(r), xt)
