"""Columns that are solved in several groups: a call that fails leaves x as it was."""
import numpy as np
import pytest
import torch

from airg_inputs import workloads

pytestmark = pytest.mark.gpu

NONFINITE = -3


@pytest.mark.parametrize("nrhs", [9, 20, 21])
def test_a_failing_column_of_a_later_group_leaves_x(nrhs):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import AirgError, Solver
    p = workloads.fv_random(700, 0.6, True, ny=640)  # solved as 8 + 1, 16 + 4, 16 + 5
    s = Solver(p.indptr, p.indices, p.data, precision=1)
    B = torch.from_numpy(p.b).cuda().repeat(nrhs, 1)
    B[nrhs - 1, 5] = float("nan")
    x = torch.rand_like(B)
    x0 = x.clone()
    with pytest.raises(AirgError) as e:
        s.solve(B, x, guess=True)
    assert e.value.code == NONFINITE
    torch.cuda.synchronize()
    assert torch.equal(x, x0)
    # a group of one column takes the single-column workspace
    B[nrhs - 1, 5] = 0.0
    X, infos = s.solve(B, x, guess=True)
    assert X is x and all(i["converged"] == 1 for i in infos)
    r = p.b - p.scipy() @ x[0].cpu().numpy()
    assert np.linalg.norm(r) <= 1e-10 * (1 + 1e-3) * np.linalg.norm(p.b)
    s.close()
