"""The smoother polynomial formed as one matrix (levels where one product with
q(A_ff) costs less than the Horner steps): which levels take it, and solves
that keep the oracle's iteration counts and solutions over the degrees, the
storage precisions and odd sizes."""
import numpy as np
import pytest
import torch

import oracle
from airg_inputs import workloads
from parity import assert_elementwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,opts", [
    ((65, 33), dict(poly_order=0)),   # nothing to form
    ((65, 33), dict(poly_order=1)),   # one product already
    ((65, 33), dict(poly_order=2)),
    ((130, 71), dict()),
    ((130, 71), dict(poly_order=6)),
    ((130, 71), dict(smooth_type=1)),
    ((130, 71), dict(smooth_type=2)),  # FCF keeps the matrix-free form
])
def test_formed_polynomial_keeps_the_oracle_solve(shape, opts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    p = workloads.fv_random(shape[0], 0.7, True, ny=shape[1])
    oracle_opts = dict(opts)
    if "smooth_type" in opts:
        oracle_opts["smooth_type"] = ("f", "fc", "fcf")[opts["smooth_type"]]
    x_o, its, _, _, _ = oracle.solve(p.scipy(), p.b, oracle.Params(**oracle_opts))
    s = Solver(p.indptr, p.indices, p.data, **opts)
    x, info = s.solve(torch.from_numpy(p.b).cuda())
    assert info["converged"] == 1 and info["iterations"] == its
    # both solve to a relative residual of 1e-10: the tolerance of the parity tests
    assert_elementwise(x.cpu().numpy(), np.asarray(x_o))
    st = s.stats()
    smoothed = st["levels"] - 1
    degrees = [d for d in st["poly_degree"][:smoothed]]
    launches = s.time_kernels("horner", 1)["launches"]
    if opts.get("smooth_type") == 2 or opts.get("poly_order", 4) < 2:
        assert launches == sum(max(d, 1) for d in degrees)
    else:
        # every level of a system this small is cheaper in one launch
        assert launches == smoothed
    s.close()


@pytest.mark.parametrize("prec", [1, 2])
def test_formed_polynomial_in_low_precision_storage(prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    p = workloads.dg_random(31, 0.5, True, ny=23)
    x_o, its, _, _, _ = oracle.solve(p.scipy(), p.b)
    s = Solver(p.indptr, p.indices, p.data, precision=prec)
    assert s.time_kernels("horner", 1)["launches"] < sum(s.stats()["poly_degree"])
    b = torch.from_numpy(p.b).cuda()
    x, info = s.solve(b)
    assert info["converged"] == 1 and info["iterations"] == its
    # x - x_o = A^{-1}(r_o - r): the dense inverse bounds it element by element
    A = p.scipy()
    r = p.b - A @ x.cpu().numpy()
    r_o = p.b - A @ np.asarray(x_o)
    inv = np.abs(np.linalg.inv(A.toarray())).sum(axis=1).max()
    bound = inv * np.abs(r - r_o).max() * (1 + 1e-6) + 1e-13 * np.abs(x_o).max()
    assert np.abs(x.cpu().numpy() - x_o).max() <= bound
    # columns take the same operator
    xs, infos = s.solve(torch.stack([b, 2 * b, b]))
    assert all(i["iterations"] == its for i in infos)
    s.close()
