"""The blocked eliminations: matrices of several 64-row classes in one launch
(up to 256 of them) or in launches of their own must give the same factor bit
for bit (no launch mixes two matrices' arithmetic), and an exact factorization
(eps = 0) over block and panel remainders solves to rounding: 1e-11 for
matrices of up to 1000 unknowns (ten times the bound of the 16x16, p = 1
grid)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2101_01763_amd as sp  # noqa: E402
from synth.dg_euler import DGConfig, make_problem  # noqa: E402


def _matrix(cfg):
    A, xs, b, _ = make_problem(cfg)
    return sp.BSRMatrix.from_numpy(A.rowptr, A.colind, A.val), xs, b


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_classes_together_and_apart(dtype):
    # 64, 128 and 128 leaves of uneven sizes: the batch's 320 go by class
    cfgs = [DGConfig(n=n, p=1, seed=n) for n in (17, 27, 31)]
    Ls = [7, 8, 8]
    mats = [_matrix(c)[0] for c in cfgs]
    Fs = sp.factor_batched([(A, c.n, c.n, True, False) for A, c in zip(mats, cfgs)], eps=1e-2, nlevels=Ls, dtype=dtype)
    for A, c, L, F in zip(mats, cfgs, Ls, Fs):
        one = sp.factor(A, c.n, c.n, True, False, eps=1e-2, nlevels=L, dtype=dtype)
        assert F.stats()["batch_systems"] == 3 and F.stats()["size_after"] == one.stats()["size_after"]
        r = torch.as_tensor(np.random.default_rng(c.n).standard_normal(c.N), device="cuda")
        assert torch.equal(F.apply(r), one.apply(r)) and torch.equal(F.apply_T(r), one.apply_T(r))


@pytest.mark.parametrize("n,p,L", [(3, 1, 1), (5, 1, 2), (5, 2, 1), (7, 1, 1), (9, 2, 3), (5, 3, 2), (12, 1, 3)])
def test_exact_sizes(n, p, L):
    cfg = DGConfig(n=n, p=p, seed=n)
    A, xs, b = _matrix(cfg)
    M = sp.factor(A, n, n, True, False, eps=0.0, nlevels=L, dtype="f64")
    x = M.apply(torch.as_tensor(b, device="cuda")).cpu().numpy()
    assert np.linalg.norm(x - xs) <= 1e-11 * np.linalg.norm(xs)
