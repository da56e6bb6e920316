"""Setup kernels that work on a matrix row per group of lanes with the row in
LDS (sorts, merges, products, drops, masked powers): matrices whose row lengths
straddle the groups' widths and capacities, up to rows too long for them, against
the oracle's hierarchy bit for bit."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import oracle
from test_gpu_parity import compare_hierarchy

pytestmark = pytest.mark.gpu


def _matrix(n, lengths, long_rows, seed):
    """Diagonally dominant, row r with lengths[r % len] entries near the diagonal,
    `long_rows` rows of a given length anywhere."""
    g = np.random.default_rng(seed)
    rows = []
    for r in range(n):
        k = min(lengths[r % len(lengths)], n)
        span = max(2 * k, 40)
        c = (r + g.choice(np.arange(-span, span), min(k, 2 * span) - 1, replace=False)) % n if k > 1 else []
        rows.append(np.unique(np.append(c, r)).astype(np.int64))
    for r, k in long_rows:
        rows[r] = np.unique(np.append(g.choice(n, k - 1, replace=False), r))
    indptr = np.concatenate([[0], np.cumsum([len(c) for c in rows])])
    indices = np.concatenate(rows)
    data = -g.random(len(indices))
    A = sp.csr_matrix((data, indices, indptr), shape=(n, n))
    A.setdiag(np.asarray(abs(A).sum(axis=1)).ravel() * (1.1 + g.random(n)) + 0.5)
    A.sort_indices()
    return A


@pytest.mark.parametrize("n,lengths,long_rows", [
    (700, (1, 2, 3, 4, 5), ()),                                  # the shortest groups
    (700, (1, 2), ((11, 16), (301, 17), (502, 31), (650, 33))),  # past the short groups' capacity
    (900, (7, 8, 9, 15, 16, 17), ((5, 63), (6, 65))),
    (1200, (30, 31, 32, 33, 64), ((77, 127), (78, 129))),
    (2500, (3, 5), ((1, 511), (900, 513), (1700, 1023), (1701, 1025), (1702, 2050))),
    (12000, (2, 3, 4), ((2000, 11000),)),                        # a row past the largest table
])
def test_hierarchy_of_uneven_rows_is_the_oracles(n, lengths, long_rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    A = _matrix(n, lengths, long_rows, 7 + n)
    opts = dict(max_levels=3, poly_order=3, coarse_poly_order=6)
    levels = oracle.setup(A, oracle.Params(**opts))
    assert len(levels) >= 2
    s = Solver(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data, keep_setup_data=1, **opts)
    compare_hierarchy(s, levels)
    x = np.random.default_rng(n).random(n)
    y, info = s.solve(torch.from_numpy(A @ x).cuda())
    assert info["converged"] == 1
    # |x - y| <= |A^{-1}| |r|, rows dominant by at least 0.5: |A^{-1}|_inf <= 2
    r = A @ x - A @ y.cpu().numpy()
    assert np.abs(x - y.cpu().numpy()).max() <= 2.0 * np.abs(r).max() + 1e-12
    s.close()
