"""Statistics of hierarchies whose polynomials are formed as one matrix: what the
complexities count, what is kept besides and what a V-cycle moves."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

from airg_inputs import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opts", [dict(), dict(poly_order=6), dict(coarse_persistent=1), dict(smoother=1),
                                  dict(max_levels=1, coarse_poly_order=8), dict(inverse_type=1)])
def test_statistics_say_what_is_counted_and_what_is_formed(opts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    p = workloads.fv_random(70, 0.6, True, ny=51)
    s = Solver(p.indptr, p.indices, p.data, keep_setup_data=1, **opts)
    st = s.stats()
    last = st["levels"] - 1
    steps = st["coarse_roots"] - 1
    cycle, kept, moved = steps * st["nnz"][last], st["nnz"][last], 0.0

    def csr(rows, nnz):
        return 12.0 * nnz + 4.0 * (rows + 1)
    n = st["n"][last]
    formed = st["nnz_formed"]
    dense = steps >= 3 and n <= 1024 and not opts.get("coarse_persistent")
    assert formed[last] == (n * n if dense else 0)
    if dense:
        moved += csr(n, n * n) + 16.0 * n
    else:
        moved += steps * (csr(n, st["nnz"][last]) + 32.0 * n)
    for l in range(last):
        L = s.export_level(l, what=("ff", "alpha"))
        nf, nc = L["n_f"], L["n_c"]
        A = sp.csr_matrix((L["ff"][2], L["ff"][1], L["ff"][0]), shape=(nf, nf))
        d = len(L["alpha"]) - 1
        if opts.get("smoother") or opts.get("inverse_type"):
            assert formed[l] == 0
        else:
            # every level of a system this small; entries that cancel to zero
            # are few and not stored
            q = sum((abs(A) ** k for k in range(1, d + 1)), sp.identity(nf, format="csr"))
            assert 0.999 * q.nnz <= formed[l] <= q.nnz
        if opts.get("smoother"):
            continue
        cycle += st["nnz_z"][l] + st["nnz_fc"][l] + (d + 1) * st["nnz_ff"][l]
        kept += st["nnz_z"][l] + st["nnz_fc"][l] + st["nnz_ff"][l]
    if not opts.get("smoother"):
        assert st["cycle_complexity"] == pytest.approx(cycle / p.nnz, rel=1e-12)
        assert st["storage_complexity"] == pytest.approx(kept / p.nnz, rel=1e-12)
    if last == 0:
        assert st["vcycle_bytes"] == pytest.approx(moved, rel=1e-12)
    elif not opts.get("inverse_type"):
        # the smoother's part is that of its launches
        assert s.time_kernels("horner", 1)["launches"] == last
    s.close()
