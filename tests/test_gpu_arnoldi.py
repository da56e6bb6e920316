"""The setup's Arnoldi process (queued without host waits, sweeps fused in the
tree order, products staged in LDS): coefficients, truncation residuals and
roots against the oracle, at sizes around the sweeps' chunks of 1024 and with
more steps than one sweep takes vectors."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import oracle
from airg_inputs import workloads
from test_gpu_parity import compare_hierarchy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,opts", [
    (32, 32, {}),                                        # 1024
    (41, 25, {}),                                        # 1025
    (33, 31, dict(poly_order=1)),                        # 1023
    (64, 67, dict(coarse_poly_order=62)),                # 63 vectors: the last in one sweep
    (64, 67, dict(coarse_poly_order=70, max_levels=2)),  # more
    (9, 8, dict(coarse_poly_order=80)),                  # as many steps as rows: breakdowns
])
def test_arnoldi_is_the_oracles(nx, ny, opts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    p = workloads.fv_random(nx, 0.6, True, ny=ny)
    levels = oracle.setup(p.scipy(), oracle.Params(**opts))
    s = Solver(p.indptr, p.indices, p.data, keep_setup_data=1, **opts)
    if opts.get("coarse_poly_order", 20) <= 20:
        compare_hierarchy(s, levels)
    else:  # long root lists are ill-conditioned: the smoother's part and the levels
        assert s.stats()["levels"] == len(levels)
        for l, L in enumerate(levels[:-1]):
            assert np.array_equal(s.export_level(l)["alpha"], L.alpha)
    s.close()


def test_breakdown_in_the_first_steps():
    # a scaled identity block next to a chain: |A v| v-parallel at once
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    n = 1500
    A = sp.csr_matrix(sp.diags([np.full(n, 2.0)], [0]))
    A.sort_indices()
    s = Solver(A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data)
    b = torch.arange(1, n + 1, dtype=torch.float64, device="cuda")
    x, info = s.solve(b)
    assert info["converged"] == 1 and torch.allclose(x, b / 2, rtol=1e-12, atol=0)
    assert s.stats()["coarse_roots"] == 1
    s.close()
