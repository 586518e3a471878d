"""stats()["factor_bytes"] against a count from the ordering: the elements of
the stored blocks that one application of M^-1 reads.  eps = 0 keeps every
unknown, so with up to two levels all sizes are those of the grid: the leaf
inverses' n^2 + e^2 (e unknowns next to the separator), each coupling block
(A_ns and A_sn), F_s and B_s of the separator's clusters, and the top's inverse
once: only the backward sweep reads it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2101_01763_amd as sp  # noqa: E402
from oracle.nd import neighbours, nested_dissection  # noqa: E402
from synth.dg_euler import DGConfig, make_problem  # noqa: E402


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n,p,L", [(4, 1, 1), (6, 1, 2), (5, 2, 2), (9, 1, 2)])
def test_count(n, p, L, dtype):
    cfg = DGConfig(n=n, p=p, seed=1)
    A, _, _, _ = make_problem(cfg)
    F = sp.factor(sp.BSRMatrix.from_numpy(A.rowptr, A.colind, A.val), n, n, True, False, eps=0.0, nlevels=L, dtype=dtype)
    nd, adj, b = nested_dissection(n, n, True, False, L), neighbours(n, n, True, False), cfg.b
    sep = {int(e) for c in nd.levels[0] if not c.interior for e in c.elems}
    count = 0
    for c in nd.levels[0]:
        m = len(c.elems) * b
        if c.interior:
            links = [sum(f in sep for f in adj[int(e)]) for e in c.elems]
            count += m * m + (np.count_nonzero(links) * b) ** 2 + 2 * sum(links) * b * b
        else:
            count += 2 * m * m
    count += (len(sep) * b) ** 2
    assert F.stats()["factor_bytes"] == count * (4 if dtype == "f32" else 8)
