"""The Newton polynomial of a small coarsest level formed as one dense matrix:
sizes around its limits and column remainders, real and complex roots, every
storage, one and several columns, against the oracle's solve."""
import numpy as np
import pytest
import torch

import oracle
from airg_inputs import workloads
from parity import assert_elementwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,order,formed", [
    (1, 3, True), (2, 3, True), (63, 2, False), (63, 3, True), (255, 8, True), (257, 9, True),
    (1023, 8, True), (1024, 9, True), (1025, 9, False)])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_one_level_matches_the_oracle(n, order, formed, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    nx = next(d for d in range(int(n ** 0.5), 0, -1) if n % d == 0)
    p = workloads.fv_random(nx, 0.4, True, ny=n // nx)
    kw = dict(max_levels=1, coarse_poly_order=order, restart=40)
    xo, its, _, _, _ = oracle.solve(p.scipy(), p.b, oracle.Params(**kw))
    s = Solver(p.indptr, p.indices, p.data, precision=prec, **kw)
    roots = s.stats()["coarse_roots"]
    # roots of a matrix of few rows are fewer than the order asks for
    launches = s.time_kernels("newton", 1)["launches"]
    if formed and roots >= 4:
        assert launches == 1
    b = torch.from_numpy(p.b).cuda()
    x, info = s.solve(b)
    assert info["converged"] == 1
    if prec == 0:
        assert info["iterations"] == its
        # both solve to a relative residual of 1e-10: the tolerance of the parity tests
        assert_elementwise(x.cpu().numpy(), np.asarray(xo))
    xs, infos = s.solve(torch.stack([b, 2 * b, b]))
    for q, i in enumerate(infos):
        assert i["converged"] == 1
        r = p.b * (1, 2, 1)[q] - p.scipy() @ xs[q].cpu().numpy()
        assert np.linalg.norm(r) <= 1e-10 * (1 + 1e-3) * np.linalg.norm(p.b) * (1, 2, 1)[q]
    s.close()
