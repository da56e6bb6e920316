"""The launch shapes operators get without the tuner: sizes on both sides of
the rule's lines, in every storage, against one lane per row."""
import numpy as np
import pytest
import torch

from airg_inputs import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [
    (3, 2),       # fewer rows than lanes
    (64, 64),     # short operators, up to 32 lanes a row
    (511, 257),   # 2^17 rows and a little at the top
    (901, 749),   # entry-staged products on level 0
])
@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("dg", [False, True])
def test_default_shapes_match_one_lane_per_row(nx, ny, prec, dg):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    if dg and nx > 512:
        nx, ny = nx // 2, ny // 2  # four points a cell
    make = workloads.dg_random if dg else workloads.fv_random
    p = make(nx, 0.6, True, ny=ny)
    # one step: x is the V-cycle of b times a scalar
    s = Solver(p.indptr, p.indices, p.data, precision=prec, max_it=1)
    b = torch.from_numpy(p.b).cuda()
    x = s.solve(b)[0].cpu().numpy()
    last = s.stats()["levels"] - 1
    for l in range(last):
        for op in ("ff", "b", "z"):
            s.set_lanes(l, op, 1)
    s.set_lanes(last, "a", 1)
    s.set_lanes(0, "top", 1)
    x1 = s.solve(b)[0].cpu().numpy()
    # the same terms summed in another order: a sum of m terms moves by at most
    # m u sum|terms|, with m below 100 in each product and about 100 products in
    # sequence in a cycle whose operators are bounded by the weights' norms
    u = 2.0 ** -53 if prec == 0 else 2.0 ** -24
    assert np.abs(x - x1).max() <= 1e4 * u * np.abs(x1).max()
    s.close()
