"""The optional formed polynomials never make a call run out of memory: where they
do not fit, the polynomials are applied step by step."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from airg_inputs import workloads
from parity import assert_elementwise

pytestmark = pytest.mark.gpu

NOMEM = -5


def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _budget(lib, nbytes):
    held = ctypes.c_int64()
    assert lib.airg_set_alloc_budget(nbytes, ctypes.byref(held)) == 0
    return held.value


def _shrinking_budgets(lib, make, launches):
    """Setups under budgets from plenty downwards until one fails: their launch
    counts and the smallest budget that one succeeded with."""
    s = make()
    limit = 4 * _budget(lib, 0)
    s.close()
    counts, smallest = [], 0
    try:
        while True:
            _budget(lib, limit)
            try:
                s = make()
            except Exception as e:  # noqa: BLE001
                assert getattr(e, "code", None) == NOMEM, e
                return counts, smallest
            counts.append(launches(s))
            s.close()
            smallest, limit = limit, int(limit * 0.985)
    finally:
        _budget(lib, 0)


@pytest.mark.parametrize("cls,opts", [
    ("horner", dict(poly_order=10)),                       # q(A_ff) of long rows
    ("newton", dict(max_levels=1, coarse_poly_order=12, restart=40)),  # the dense coarsest polynomial
])
def test_a_setup_that_cannot_hold_the_formed_polynomials_keeps_the_steps(cls, opts):
    _needs_gpu()
    from paper_2508_17517_amd import Solver, binding
    lib = binding.load()
    p = workloads.fv_random(32, 0.7, True) if cls == "newton" else workloads.fv_random(64, 0.7, True)
    xo, its, _, _, _ = oracle.solve(p.scipy(), p.b, oracle.Params(**opts))

    def make():
        return Solver(p.indptr, p.indices, p.data, **opts)
    counts, limit = _shrinking_budgets(lib, make, lambda s: s.time_kernels(cls, 1)["launches"])
    # with less memory the polynomial is applied step by step, before the setup fails
    assert counts[-1] > counts[0], counts
    _budget(lib, limit)
    try:
        s = make()
        assert s.time_kernels(cls, 1)["launches"] == counts[-1]
    finally:
        _budget(lib, 0)
    x, info = s.solve(torch.from_numpy(p.b).cuda())
    assert info["converged"] == 1 and info["iterations"] == its
    assert_elementwise(x.cpu().numpy(), np.asarray(xo))
    s.close()


@pytest.mark.parametrize("graph", [0, 1])
def test_a_later_workspace_takes_the_formed_polynomials_memory(graph):
    # one right-hand side, then several: where the columns' workspace does not
    # fit beside the formed polynomials, they go and the solve runs without
    _needs_gpu()
    from paper_2508_17517_amd import Solver, binding
    lib = binding.load()
    p = workloads.fv_random(64, 0.7, True)
    opts = dict(poly_order=10, restart=4, graph=graph)
    xo, its, _, _, _ = oracle.solve(p.scipy(), p.b, oracle.Params(poly_order=10, restart=4))
    s = Solver(p.indptr, p.indices, p.data, **opts)
    formed = s.time_kernels("horner", 1)["launches"]
    b = torch.from_numpy(p.b).cuda()
    x0, _ = s.solve(b)
    one = _budget(lib, 0)
    X, _ = s.solve(torch.stack([b, b]))
    need = _budget(lib, 0) - one
    s.trim()
    _budget(lib, one + need // 2)
    try:
        X, infos = s.solve(torch.stack([b, b]))
    finally:
        _budget(lib, 0)
    assert s.time_kernels("horner", 1)["launches"] > formed
    x, info = s.solve(b)
    for y, i in ((X[0], infos[0]), (X[1], infos[1]), (x, info)):
        assert i["converged"] == 1 and i["iterations"] == its
        assert_elementwise(y.cpu().numpy(), np.asarray(xo))
    s.close()
