"""A^T x without a transposed copy, against NumPy: block sizes on both sides of
the line between one lane per row and one wave per element, rows of more than
64 blocks (the mirrors are searched 64 at a time), values off 16-byte
alignment, and the outer product on the pattern.  Sums of n products in FP64:
within n eps (|A|^T |x|)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2101_01763_amd as sp  # noqa: E402


def _arrow(n, bs, seed):
    """Tridiagonal blocks plus a full first block row and column."""
    rng = np.random.default_rng(seed)
    cols = [np.arange(n)] + [np.unique(np.clip([0, i - 1, i, i + 1], 0, n - 1)) for i in range(1, n)]
    rowptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    colind = np.concatenate(cols).astype(np.int32)
    return rowptr, colind, rng.standard_normal((len(colind), bs, bs))


@pytest.mark.parametrize("bs", [2, 4, 8, 10, 12, 16, 22, 34, 36, 62, 64])
@pytest.mark.parametrize("n,off", [(1, 0), (7, 0), (70, 0), (130, 1)])
def test_transposed_product(bs, n, off):
    rowptr, colind, val = _arrow(n, bs, 100 * n + bs)
    A = sp.BSRMatrix.from_numpy(rowptr, colind, val)
    flat = torch.as_tensor(val, device="cuda").reshape(-1)
    buf = torch.empty(flat.numel() + off, dtype=torch.float64, device="cuda")
    buf[off:] = flat
    v = buf[off:].reshape(val.shape)
    rng = np.random.default_rng(n)
    x, y = rng.standard_normal((2, n * bs))
    ref, mag, cnt = np.zeros(n * bs), np.zeros(n * bs), np.zeros(n * bs)
    for i in range(n):
        for t in range(rowptr[i], rowptr[i + 1]):
            J = slice(colind[t] * bs, (colind[t] + 1) * bs)
            xi = x[i * bs:(i + 1) * bs]
            ref[J] += val[t].T @ xi
            mag[J] += np.abs(val[t]).T @ np.abs(xi)
            cnt[J] += bs
    out = sp.spmv(A, torch.as_tensor(x, device="cuda"), transpose=True, alpha=-0.5, beta=2.0,
                  y=torch.as_tensor(y, device="cuda"), val=v).cpu().numpy()
    eps = np.finfo(float).eps
    assert np.all(np.abs(out - (2.0 * y - 0.5 * ref)) <= eps * ((cnt + 2) * mag + 4.0 * np.abs(y)))
    po = sp.pattern_outer(A, torch.as_tensor(x, device="cuda"), torch.as_tensor(y, device="cuda"), alpha=3.0).cpu().numpy()
    xb, yb = x.reshape(n, bs), y.reshape(n, bs)
    rows = np.repeat(np.arange(n), np.diff(rowptr))
    assert np.array_equal(po, (3.0 * xb[rows])[:, :, None] * yb[colind][:, None, :])
