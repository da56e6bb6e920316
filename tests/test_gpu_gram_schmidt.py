"""The two Gram-Schmidt sweeps of a step at the sizes where the partial sums
move from the next sweep into launches of their own, against the sweeps of
interleaved columns."""
import numpy as np
import pytest
import torch

from airg_inputs import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(2, 1), (32, 32), (41, 25), (256, 256), (257, 256)])
@pytest.mark.parametrize("steps", [2, 6])
@pytest.mark.parametrize("lookahead", [0, 1])
def test_sweeps_match_those_of_columns(nx, ny, steps, lookahead):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    p = workloads.fv_random(nx, 0.5, True, ny=ny)
    s = Solver(p.indptr, p.indices, p.data, max_it=steps, lookahead=lookahead)
    b = torch.from_numpy(p.b).cuda()
    x, info = s.solve(b)
    X, infos = s.solve(torch.stack([b, b]))
    assert infos[0]["iterations"] == info["iterations"]
    x = x.cpu().numpy()
    # sums of the same terms in another order, through the cycles of the steps:
    # below 100 terms and about 100 products in sequence in each
    tol = 1e4 * steps * 2.0 ** -53 * np.abs(x).max()
    assert np.abs(X[0].cpu().numpy() - x).max() <= tol
    x2 = s.solve(b)[0].cpu().numpy()
    assert np.array_equal(x2, x)
    s.close()
