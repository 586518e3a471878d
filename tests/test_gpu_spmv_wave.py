"""y = A x with one wave per element (bs = 16 and 36, values on 16-byte
boundaries) and by lane groups (other sizes, other alignments) against NumPy:
rows of one, of a few and of many blocks, an element count off the workgroup's
four.  Sums of n products in FP64: within n eps (|A| |x|)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2101_01763_amd as sp  # noqa: E402


@pytest.mark.parametrize("bs", [4, 16, 36, 64])
@pytest.mark.parametrize("n,off", [(1, 0), (7, 0), (70, 0), (130, 1)])
def test_product(bs, n, off):
    rng = np.random.default_rng(10 * n + bs)
    cols = [np.arange(n)] + [np.unique(np.clip([0, i - 1, i, i + 1], 0, n - 1)) for i in range(1, n)]
    rowptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])])
    colind = np.concatenate(cols)
    val = rng.standard_normal((len(colind), bs, bs))
    x, y = rng.standard_normal((2, n * bs))
    A = sp.BSRMatrix.from_numpy(rowptr, colind, val)
    buf = torch.empty(val.size + off, dtype=torch.float64, device="cuda")
    v = buf[off:].reshape(val.shape)
    v.copy_(A.val)
    out = sp.spmv(A, torch.as_tensor(x, device="cuda"), alpha=-0.5, beta=2.0, y=torch.as_tensor(y, device="cuda"),
                  val=v).cpu().numpy()
    rows = np.repeat(np.arange(n), np.diff(rowptr))
    ref, mag = np.zeros((2, n, bs))
    np.add.at(ref, rows, np.einsum("trc,tc->tr", val, x.reshape(n, bs)[colind]))
    np.add.at(mag, rows, np.einsum("trc,tc->tr", np.abs(val), np.abs(x.reshape(n, bs)[colind])))
    terms = np.diff(rowptr)[:, None] * bs + 2
    err = np.abs(out.reshape(n, bs) - (2.0 * y.reshape(n, bs) - 0.5 * ref))
    assert np.all(err <= np.finfo(float).eps * (terms * mag + 4.0 * np.abs(y.reshape(n, bs))))
