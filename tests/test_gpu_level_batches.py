"""Sweeps whose clusters have more inputs than one workgroup stages at a time:
separators coupled to every separator above and below them in the ordering give
a cluster more than LEVEL_MAXIT neighbours or more than LEVEL_CAP inputs, which
are then taken in several batches.  The ordering says on the CPU that both
sweeps have such a cluster.  36x36 with 4 unknowns an element: neighbours'
products recomputed in the workgroup; 28x28 with 36: couplings and own matrix in
one launch (FP32, 254 KB) and bands of rows (FP64).

eps = 0 is an exact factorization and the operator is within 1/2 of 2 I (norm),
so M^-1 (A x) = x up to the rounding of eliminations of up to 1008 unknowns over
10 levels: 1e-11 in FP64; in FP32 n u = 6e-5 for the largest matrix, 1e-3 with
the levels.  M^-T is the exact transpose of M^-1 as stored: the products' FP64
sums of up to 3600 terms over 10 levels, 1e-12 of the norms."""
import os
import re

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2101_01763_amd as sp  # noqa: E402
from oracle.nd import neighbours, nested_dissection  # noqa: E402


def _limit(name):
    src = open(os.path.join(os.path.dirname(sp.__file__), "csrc", "internal.h")).read()
    return int(re.search(rf"constexpr int {name} = (\d+);", src)[1])


def _batches(sizes):
    cap, most = _limit("LEVEL_CAP"), _limit("LEVEL_MAXIT")
    n, first, off = 1, 0, 0
    for i, k in enumerate(sizes):
        if i > first and (off + k > cap or i - first == most):
            n, first, off = n + 1, i, 0
        off += k
    return n


def _above(a, b):
    """Whether node a lies above node b in the tree (heap numbers)."""
    while b > a:
        b >>= 1
        if a == b:
            return True
    return False


def _operator(nx, ny, bs, nd):
    node = nd.node_of_elem
    seps = np.array([e for e in range(nx * ny) if nd.node_level[int(node[e])] > 0])
    cols = [set(q) | {e} for e, q in enumerate(neighbours(nx, ny, False, False))]
    for k in {int(q) for q in node[seps]}:
        mine = seps[node[seps] == k]
        kin = [int(e) for e in seps if node[e] == k or _above(int(node[e]), k) or _above(k, int(node[e]))]
        for e in mine:
            cols[int(e)].update(kin)
    cols = [sorted(c) for c in cols]
    rowptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    colind = np.concatenate(cols).astype(np.int32)
    width = max(len(c) for c in cols) * bs
    gen = torch.Generator(device="cuda")
    gen.manual_seed(nx)
    # a random matrix of at most `width` entries a row and column has norm 2 sqrt(width)
    val = torch.randn(len(colind), bs, bs, generator=gen, dtype=torch.float64, device="cuda") / (4.0 * width ** 0.5)
    rows = np.repeat(np.arange(nx * ny), np.diff(rowptr))
    val[torch.as_tensor(rows == colind, device="cuda")] += 2.0 * torch.eye(bs, dtype=torch.float64, device="cuda")
    return sp.BSRMatrix(torch.as_tensor(rowptr, device="cuda"), torch.as_tensor(colind, device="cuda"), val)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,bs,L", [(36, 4, 10), (28, 36, 6)])
def test_several_batches(n, bs, L, dtype):
    nd = nested_dissection(n, n, False, False, L)
    fwd = bwd = 0
    for cl in nd.levels[1:]:
        ints, ifs = [c for c in cl if c.interior], [c for c in cl if not c.interior]
        fwd = max([fwd] + [_batches([len(s.elems) * bs for s in ints if _above(f.node, s.node)]) for f in ifs])
        bwd = max([bwd] + [_batches([len(f.elems) * bs for f in ifs if _above(f.node, s.node)]) for s in ints])
    assert fwd >= 2 and bwd >= 2
    A = _operator(n, n, bs, nd)
    M = sp.factor(A, n, n, False, False, eps=0.0, nlevels=L, dtype=dtype)
    rng = np.random.default_rng(n)
    u, v = (torch.as_tensor(rng.standard_normal(A.N), device="cuda") for _ in range(2))
    Mu, Mtv = M.apply(u), M.apply_T(v)
    assert abs(Mu @ v - u @ Mtv) <= 1e-12 * Mu.norm() * v.norm()
    tol = 1e-11 if dtype == "f64" else 1e-3
    assert (M.apply(sp.spmv(A, u)) - u).norm() <= tol * u.norm()
    assert (M.apply_T(sp.spmv(A, v, transpose=True)) - v).norm() <= tol * v.norm()
    assert torch.equal(M.apply(u), Mu) and torch.equal(M.apply_T(v), Mtv)
    E = sp.factor(A, n, n, False, False, eps=0.0, nlevels=L, dtype=dtype, graphs=False)
    assert torch.equal(E.apply(u), Mu) and torch.equal(E.apply_T(v), Mtv)
