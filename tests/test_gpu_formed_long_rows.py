"""Small levels whose formed polynomial has long rows: one product streams them
faster than the steps' launches take."""
import pytest
import torch

from airg_inputs import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_small_levels_with_long_rows_are_formed(prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    p = workloads.fv_random(512, 0.3, True)
    s = Solver(p.indptr, p.indices, p.data, precision=prec)
    st = s.stats()
    levels = st["levels"] - 1
    launches = s.time_kernels("horner", 1)["launches"]
    s.close()
    # level 4: 11,497 rows of 198 entries; the last one 6,409 of 303
    assert levels == 6
    assert launches == levels
