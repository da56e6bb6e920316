"""Interleaved columns: products whose rows are shared by several lanes, over
the column counts and sizes where the split changes, against one column."""
import numpy as np
import pytest
import torch

from airg_inputs import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(3, 2), (64, 64), (301, 217)])
@pytest.mark.parametrize("nrhs", [2, 3, 8, 33, 64])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_columns_match_one_column(nx, ny, nrhs, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    p = workloads.fv_random(nx, 0.6, True, ny=ny)
    # one step: x is the V-cycle of b times a scalar
    s = Solver(p.indptr, p.indices, p.data, precision=prec, max_it=1)
    rng = np.random.default_rng(nrhs)
    B = torch.from_numpy(p.b[None, :] * rng.uniform(0.5, 1.5, (nrhs, p.n))).cuda()
    X = s.solve(B)[0].cpu().numpy()
    # the same terms summed in another order: a sum of m terms moves by at most
    # m u sum|terms|, with m below 100 in each product and about 100 products in
    # sequence in a cycle whose operators are bounded by the weights' norms
    u = 2.0 ** -53 if prec == 0 else 2.0 ** -24
    for c in sorted({0, 1, nrhs // 2, nrhs - 1}):
        x = s.solve(B[c])[0].cpu().numpy()
        assert np.abs(X[c] - x).max() <= 1e4 * u * np.abs(x).max()
    s.close()


@pytest.mark.parametrize("nrhs", [5, 9, 20])
@pytest.mark.parametrize("guess", [False, True])
def test_columns_split_over_solves(nrhs, guess):
    # large enough that 9 and 20 columns are solved as 8 + 1 and 16 + 4
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    p = workloads.fv_random(700, 0.6, True, ny=640)
    s = Solver(p.indptr, p.indices, p.data)
    rng = np.random.default_rng(nrhs)
    B = torch.from_numpy(p.b[None, :] * rng.uniform(0.5, 1.5, (nrhs, 1))).cuda()
    X0 = torch.zeros_like(B)
    X0[::2] = 1.0
    X, infos = s.solve(B, X0.clone(), guess=True) if guess else s.solve(B)
    assert len(infos) == nrhs
    A = p.scipy()
    for c in range(nrhs):
        x, info = s.solve(B[c], X0[c].clone(), guess=True) if guess else s.solve(B[c])
        assert infos[c]["converged"] == 1 and infos[c]["iterations"] == info["iterations"]
        b = B[c].cpu().numpy()
        # the default tolerance, and the rounding of forming the residual here
        assert np.linalg.norm(b - A @ X[c].cpu().numpy()) <= 1e-10 * (1 + 1e-3) * np.linalg.norm(b)
    s.close()
