"""The smoother under BF16 storage keeps the precision of the steps: BF16 copies
of A_ff with FP32 coefficients, on the systems where rounding the polynomial's
own entries to BF16 would lose most."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

from airg_inputs import workloads

pytestmark = pytest.mark.gpu


def _bf16(v):
    b = np.asarray(v, np.float32).view(np.uint32)
    return ((b + 0x7FFF + ((b >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32).astype(np.float64)


def _q(A, alpha, s):
    y = alpha[-1] * s
    for a in alpha[-2::-1]:
        y = A @ y + a * s
    return y


@pytest.mark.parametrize("theta", [0.1, 0.3, 0.7, 1.1, 1.3])
@pytest.mark.parametrize("level", [0, 1, 2])
def test_bf16_smoother_is_as_close_as_the_steps(theta, level):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import BF16, Solver
    p = workloads.fv_random(96, theta, True)
    s = Solver(p.indptr, p.indices, p.data, keep_setup_data=1)
    L = s.export_level(level)
    if level == 0:
        L["a"] = (p.indptr, p.indices, p.data)
    s.close()
    nf, nc = L["n_f"], L["n_c"]
    ff = sp.csr_matrix((L["ff"][2], L["ff"][1], L["ff"][0]), shape=(nf, nf))

    def empty(rows):
        return np.zeros(rows + 1, np.int32), np.zeros(0, np.int32), np.zeros(0)
    # F and C points apart from each other: with b = 0 on the C points one V-cycle
    # is q(A_ff) b_F, and one FGMRES step a multiple of it
    eye = (np.arange(nc + 1, dtype=np.int32), np.arange(nc, dtype=np.int32), np.ones(nc))
    h = Solver.from_hierarchy(
        [dict(state=L["state"], a=L["a"], ff=L["ff"], fc=empty(nf), z=empty(nc),
              cmap=np.full(nf, -1, np.int32), alpha=L["alpha"]),
         dict(a=eye, roots=np.array([1.0 + 0j]))], precision=BF16, max_it=1)
    F = np.flatnonzero(L["state"] == 1)
    rng = np.random.default_rng(7)
    b = np.zeros(nf + nc)
    # BF16 numbers, so that the vectors' own FP32 rounding stays below
    b[F] = _bf16(rng.uniform(0.5, 1.5, nf))
    x = h.solve(torch.from_numpy(b).cuda())[0].cpu().numpy()[F]
    h.close()
    exact = _q(ff, L["alpha"], b[F])
    low = ff.copy()
    low.data = _bf16(ff.data)
    steps = _q(low, L["alpha"], b[F])

    def err(y):  # off the exact direction
        y = y * (y @ exact) / (y @ y)
        return np.linalg.norm(y - exact) / np.linalg.norm(exact)
    # FP32 vectors, coefficients and sums: at most 20 roundings deep
    assert err(x) <= err(steps) + 20 * 2.0 ** -24
