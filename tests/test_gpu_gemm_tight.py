"""FP32 products against FP64 where a wrong fourth digit shows: operators
within 1/2 of 2 I (norm) have no growth to speak of, so an exact factorization
(eps = 0) in FP32 differs from the FP64 one by the rounding of its steps alone.
A step (inverse, Schur product, LU, inverse of U, scaling, QR, its completion,
two compressions, F and B: at most ten a level) on a matrix of n <= 1024
unknowns loses sqrt(n) u = 2e-6 of the largest entry; three levels add up to
6e-5, taken in the largest error of any entry.  Sizes leave remainders of the
64-row tiles, the 32-deep chunks, the 64-column blocks and the 16-byte loads."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2101_01763_amd as sp  # noqa: E402
from oracle.nd import neighbours  # noqa: E402


@pytest.mark.parametrize("nx,ny,bs,L", [(1, 1, 2, 1), (3, 1, 14, 1), (5, 1, 26, 1), (4, 4, 62, 1), (7, 5, 18, 2),
                                        (9, 7, 10, 3), (13, 11, 6, 3), (16, 16, 2, 3), (8, 12, 22, 3), (6, 6, 50, 3)])
def test_f32_is_f64_to_five_digits(nx, ny, bs, L):
    K = nx * ny
    cols = [sorted({e, *q}) for e, q in enumerate(neighbours(nx, ny, False, False))]
    rowptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    colind = np.concatenate(cols).astype(np.int32)
    rng = np.random.default_rng(bs)
    val = rng.standard_normal((len(colind), bs, bs)) / (4.0 * np.sqrt(5 * bs))   # norm 2 sqrt(5 bs) / (4 sqrt(5 bs))
    val[np.repeat(np.arange(K), np.diff(rowptr)) == colind] += 2.0 * np.eye(bs)
    A = sp.BSRMatrix.from_numpy(rowptr, colind, val)
    r = torch.as_tensor(rng.standard_normal(A.N), device="cuda")
    F, G = (sp.factor(A, nx, ny, False, False, eps=0.0, nlevels=L, dtype=t) for t in ("f32", "f64"))
    for x, y in ((F.apply(r), G.apply(r)), (F.apply_T(r), G.apply_T(r))):
        assert float((x - y).abs().max()) <= 6e-5 * float(y.abs().max())
