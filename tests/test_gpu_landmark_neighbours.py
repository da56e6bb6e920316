"""The locality order where a landmark's region touches more others than its table
holds: the order falls back to the distances of the top graph, and the hierarchy
and its solve are the oracle's."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import oracle
from airg_inputs import workloads
from parity import assert_elementwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entries", [20, 400])
def test_a_row_that_reaches_everywhere(entries):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    p = workloads.fv_random(100, 0.6, True)
    rng = np.random.default_rng(entries)
    i = 4321
    row = sp.csr_matrix((-rng.uniform(0.5, 1.0, entries) / entries,
                         (np.full(entries, i), rng.choice(p.n, entries, replace=False))), shape=(p.n, p.n))
    A = sp.csr_matrix(p.scipy() + row)
    A.sort_indices()
    xo, its, _, _, _ = oracle.solve(A, p.b)
    s = Solver(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data)
    x, info = s.solve(torch.from_numpy(p.b).cuda())
    assert info["converged"] == 1 and info["iterations"] == its
    # both solve to a relative residual of 1e-10: the tolerance of the parity tests
    assert_elementwise(x.cpu().numpy(), np.asarray(xo))
    s.close()
