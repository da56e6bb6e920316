"""Pinning launch shapes on levels whose smoother is one product with the formed
polynomial: whatever the tuner may choose for that matrix can be pinned."""
import numpy as np
import pytest
import torch

from airg_inputs import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
def test_shapes_of_the_formed_smoother_can_be_pinned(prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import AirgError, Solver
    p = workloads.fv_random(130, 0.7, True, ny=71)
    # one step: x is the V-cycle of b times a scalar
    s = Solver(p.indptr, p.indices, p.data, precision=prec, max_it=1)
    st = s.stats()
    b = torch.from_numpy(p.b).cuda()
    smoothed = st["levels"] - 1
    assert s.time_kernels("horner", 1)["launches"] == smoothed  # all formed
    x0 = s.solve(b)[0].cpu().numpy()
    u = 2.0 ** -53 if prec == 0 else 2.0 ** -24
    rows_only = 0
    for l in range(smoothed):
        ff = st["nnz_ff"][l] / st["n_f"][l]
        for lanes, lds in [(0, 0), (1, 0), (64, 0), (1, 2)] + [(k, 1) for k in (2, 4, 8, 16)]:
            try:
                s.set_lanes(l, "ff", lanes, 1, lds)
            except AirgError:
                # row blocks are made from 8 entries a row on; q(A_ff) has
                # more than A_ff, so the shape has to be refused only below that
                assert lanes == 0 and ff < 4, (l, ff, lanes, lds)
                continue
            rows_only += lanes == 0 and ff < 8
            x = s.solve(b)[0].cpu().numpy()
            # the same terms in another order: below 100 terms a sum in each of
            # about 100 products in sequence
            assert np.abs(x - x0).max() <= 1e4 * u * np.abs(x0).max()
    assert rows_only > 0  # a level whose row blocks are those of the polynomial
    s.close()


def test_tuned_shapes_pin_and_read_back():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    p = workloads.fv_random(130, 0.7, True, ny=71)
    s = Solver(p.indptr, p.indices, p.data)
    shapes = s.autotune(2)
    b = torch.from_numpy(p.b).cuda()
    x = s.solve(b)[0]
    t = Solver(p.indptr, p.indices, p.data)
    t.pin_shapes(shapes)
    assert torch.equal(t.solve(b)[0], x)
    # the tuner's defaults are the shapes in force
    for a, c in zip(shapes, t.autotune(1)):
        assert (a["level"], a["op"]) == (c["level"], c["op"])
        assert (a["lanes"], a["xcd_map"], a["lds"]) == (
            c["default_lanes"], c["default_xcd_map"], c["default_lds"]), a
    s.close()
    t.close()
