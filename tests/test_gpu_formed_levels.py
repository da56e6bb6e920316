"""Which levels' smoother polynomials are formed as one matrix: those where one
product costs less in a solve than the steps do."""
import pytest
import torch

from airg_inputs import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec,formed", [
    (512, 0, (0, 1, 2, 3)),  # launches are most of a product
    (2048, 0, (0, 1)),       # level 2: 47 us in one product, 44 in its four steps
    (2048, 1, (0, 1)),
    (2048, 2, (0, 1)),
])
def test_levels_whose_polynomial_is_formed(n, prec, formed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    p = workloads.fv_random(n, 0.3, True)
    s = Solver(p.indptr, p.indices, p.data, precision=prec)
    st = s.stats()
    degrees = st["poly_degree"][:st["levels"] - 1]
    launches = s.time_kernels("horner", 1)["launches"]
    s.close()
    if n == 512:  # at least these
        assert launches <= sum(1 if l in formed else d for l, d in enumerate(degrees))
    else:
        assert launches == sum(1 if l in formed else d for l, d in enumerate(degrees))
