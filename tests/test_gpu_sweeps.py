"""The sweeps of M^-1 and M^-T over every way a level is launched: steps
fused (matrices up to 64 KB), couplings and own matrix together (up to 256
KB), bands of rows (larger), inputs of a cluster in one staged batch or
several; unit, odd and vector-multiple cluster sizes.  eps = 0 keeps every
unknown, so the upper levels' clusters grow to the separators' full size.

Tolerances.  eps = 0 is an exact factorization: M^-1 (A x) = x up to the
rounding of the elimination, 1e-11 for leaves and separators of up to 1000
unknowns (ten times the bound of the 16x16, p = 1 grid).  M^-T is the exact
transpose of M^-1 as stored: <M^-1 u, v> and <u, M^-T v> differ by the
rounding of at most 8 products per level, sqrt(n) u each, against the norms:
1e-12 |M^-1 u| |v| covers n = 2048 over 10 levels 10 times."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2101_01763_amd as sp  # noqa: E402
from synth.dg_euler import DGConfig, make_problem  # noqa: E402


@pytest.mark.parametrize("n,p,L,eps,dtype", [
    (6, 1, 4, 0.0, "f64"), (13, 2, 5, 0.0, "f64"), (8, 3, 4, 0.0, "f64"), (24, 1, 6, 0.0, "f64"),
    (6, 1, 4, 1e-2, "f32"), (13, 2, 5, 1e-2, "f32"), (18, 3, 6, 1e-2, "f32"), (8, 3, 4, 0.0, "f32"),
    (18, 3, 6, 1e-2, "f64"), (24, 1, 6, 1e-1, "f64"), (32, 2, 8, 1e-3, "f32")])
def test_sweeps(n, p, L, eps, dtype):
    cfg = DGConfig(n=n, p=p, seed=n + p)
    A, xs, b, _ = make_problem(cfg)
    dA = sp.BSRMatrix.from_numpy(A.rowptr, A.colind, A.val)
    M = sp.factor(dA, n, n, True, False, eps=eps, nlevels=L, dtype=dtype)
    Me = sp.factor(dA, n, n, True, False, eps=eps, nlevels=L, dtype=dtype, graphs=False)
    rng = np.random.default_rng(n)
    u, v = (torch.as_tensor(rng.standard_normal(cfg.N), device="cuda") for _ in range(2))
    Mu, Mtv = M.apply(u), M.apply_T(v)
    assert abs(Mu @ v - u @ Mtv) <= 1e-12 * Mu.norm() * v.norm()
    assert torch.equal(Mu, Me.apply(u)) and torch.equal(Mtv, Me.apply_T(v))
    w = u.clone()
    M.apply(w, out=w)                        # in place, and again on warm buffers
    assert torch.equal(w, Mu)
    if eps == 0.0 and dtype == "f64":
        dx, db = torch.as_tensor(xs, device="cuda"), torch.as_tensor(b, device="cuda")
        dbt = torch.as_tensor(A.to_scipy().T @ xs, device="cuda")
        assert (M.apply(db) - dx).norm() <= 1e-11 * dx.norm()
        assert (M.apply_T(dbt) - dx).norm() <= 1e-11 * dx.norm()
