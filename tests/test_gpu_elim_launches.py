"""Fused eliminations of more than 256 matrices in several 64-row classes, the
largest class between others: the classes before and after it that are at most
256 together share a launch, more than 256 keep theirs.  The launches never mix
two matrices' arithmetic, so every system of such a batch has the factor it has
alone, bit for bit.  One level: the whole system is one matrix (Gauss-Jordan);
two levels: one separator, 2 ny elements (LU, inverse of U, completion of Q)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2101_01763_amd as sp  # noqa: E402

BS = 16


def _matrix(nx, ny):
    """Five-point blocks, periodic in x, dominated by the diagonal."""
    rng = np.random.default_rng(100 * nx + ny)
    cols = []
    for e in range(nx * ny):
        i, j = e % nx, e // nx
        cols.append(sorted({e, j * nx + (i + 1) % nx, j * nx + (i - 1) % nx}
                           | {e + d for d, ok in ((nx, j + 1 < ny), (-nx, j > 0)) if ok}))
    rowptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    colind = np.concatenate(cols).astype(np.int32)
    val = rng.standard_normal((len(colind), BS, BS)) / BS
    val[np.repeat(np.arange(nx * ny), np.diff(rowptr)) == colind] += 2.0 * np.eye(BS)
    return sp.BSRMatrix.from_numpy(rowptr, colind, val)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("L,counts", [
    # 512 and 448 rows | 270 of 384 | 256, 128, 64 and 48
    (1, {(8, 4): 1, (7, 4): 5, (6, 4): 270, (4, 4): 30, (4, 2): 20, (2, 2): 10, (3, 1): 9}),
    # 512 | 260 of 384 | 260 of 128 and ten of 64: more than 256 after the largest class
    (1, {(8, 4): 1, (6, 4): 260, (4, 2): 260, (2, 2): 10}),
    # separators of 512 and 384 rows | 270 of 256 | 192, 128 and 64
    (2, {(16, 16): 1, (12, 12): 3, (8, 8): 270, (6, 6): 20, (4, 4): 20, (2, 2): 15}),
])
def test_as_alone(L, counts, dtype):
    mats = {g: _matrix(*g) for g in counts}
    order = [g for g, k in counts.items() for _ in range(k)]
    np.random.default_rng(L).shuffle(order)
    order = [tuple(int(q) for q in g) for g in order]
    Fs = sp.factor_batched([(mats[g], *g, True, False) for g in order], eps=1e-2, nlevels=L, dtype=dtype)
    assert all(F.stats()["batch_systems"] == len(order) > 256 for F in Fs[:1])
    want = {}
    for g, A in mats.items():
        r = torch.as_tensor(np.random.default_rng(A.N).standard_normal(A.N), device="cuda")
        one = sp.factor(A, *g, True, False, eps=1e-2, nlevels=L, dtype=dtype)
        want[g] = r, one.apply(r), one.apply_T(r)
        assert torch.isfinite(want[g][1]).all()
    for g, F in zip(order, Fs):
        r, x, xt = want[g]
        assert torch.equal(F.apply(r), x) and torch.equal(F.apply_T(r), xt), g
