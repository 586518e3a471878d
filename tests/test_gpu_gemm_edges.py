"""FP32 products whose rows, columns and depths leave remainders of the 64-row
tiles and the 32-deep chunks: an exact factorization (eps = 0) in FP32 is the
FP64 one up to the rounding of eliminations of up to 1000 unknowns: n eps32 =
6e-5, with a growth of up to 16 on these well-conditioned operators, 1e-3."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2101_01763_amd as sp  # noqa: E402
from synth.dg_euler import DGConfig, make_problem  # noqa: E402


@pytest.mark.parametrize("n,p,L", [(3, 1, 1), (5, 1, 2), (5, 2, 1), (7, 1, 1), (9, 2, 3), (5, 3, 2), (12, 1, 3)])
def test_exact_f32(n, p, L):
    cfg = DGConfig(n=n, p=p, seed=n)
    A, _, b, _ = make_problem(cfg)
    mat = sp.BSRMatrix.from_numpy(A.rowptr, A.colind, A.val)
    r = torch.as_tensor(b, device="cuda")
    F, G = (sp.factor(mat, n, n, True, False, eps=0.0, nlevels=L, dtype=t) for t in ("f32", "f64"))
    for x, y in ((F.apply(r), G.apply(r)), (F.apply_T(r), G.apply_T(r))):
        assert torch.isfinite(x).all() and float((x - y).norm()) <= 1e-3 * float(y.norm())
