"""The locality order from landmarks (the coarsest points): a renumbering, so
solves keep the iteration count and the solution of the unordered solve at the
sizes where the sort's blocks and the coarsest level's graph begin and end."""
import numpy as np
import pytest
import torch

from airg_inputs import workloads
from parity import assert_elementwise

pytestmark = pytest.mark.gpu


def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("nx,ny,theta", [
    (9, 9, 0.3),         # the coarsest level is the top or nearly so
    (95, 43, 0.3),       # 4085 unknowns: one block of the sort
    (64, 64, 0.3),       # 4096
    (128, 65, 1.2),      # 8320: more than two blocks
    (2, 3000, 0.7),      # thin and deep
    (3000, 2, 0.7),
    (70, 60, 0.0),       # grid lines: not connected
    (181, 179, 0.785),
])
def test_order_keeps_the_solve(nx, ny, theta):
    _needs_gpu()
    from paper_2508_17517_amd import Solver
    p = workloads.fv_random(nx, theta, True, ny=ny)
    b = torch.from_numpy(p.b).cuda()
    got = []
    for order in (0, 1):
        s = Solver(p.indptr, p.indices, p.data, locality_order=order)
        x, info = s.solve(b)
        x2, _ = s.solve(b)
        assert info["converged"] == 1 and torch.equal(x, x2)
        got.append((x.cpu().numpy(), info["iterations"]))
        s.close()
    assert got[0][1] == got[1][1]
    assert_elementwise(got[1][0], got[0][0])
    # the order itself does not depend on the run
    s = Solver(p.indptr, p.indices, p.data)
    x, _ = s.solve(b)
    assert np.array_equal(x.cpu().numpy(), got[1][0])
    s.close()


@pytest.mark.parametrize("count", [2, 40])
def test_order_of_a_batch_with_tiny_problems(count):
    _needs_gpu()
    from paper_2508_17517_amd import BatchSolver, Solver
    probs = [workloads.fv_random(n, 0.4 + 0.01 * q, True, ny=m, seed=400 + q)
             for q, (n, m) in enumerate([(1, 1), (33, 20), (2, 2), (64, 31)] * (count // 2))][:max(count, 4)]
    mats = [(p.indptr, p.indices, p.data) for p in probs]
    got = []
    for order in (0, 1):
        s = BatchSolver(mats, locality_order=order)
        xs, infos = s.solve([torch.from_numpy(p.b).cuda() for p in probs])
        assert all(i["converged"] == 1 for i in infos)
        got.append([x.cpu().numpy() for x in xs])
        s.close()
    for p, x0, x1 in zip(probs, *got):
        # |x - u| <= |A^{-1}| rtol |b|, the same bound for both
        A = p.scipy()
        inv = np.abs(np.linalg.inv(A.toarray())).sum(axis=1).max()
        for x in (x0, x1):
            r = np.abs(p.b - A @ x).max()
            assert np.linalg.norm(p.b - A @ x) <= 1.0001e-10 * np.linalg.norm(p.b)
            assert np.abs(x - np.linalg.solve(A.toarray(), p.b)).max() <= inv * r + 1e-12
