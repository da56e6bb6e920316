"""V-cycles of integer hierarchies: every product is exact in FP64, FP32 and BF16
storage, so the default launch shapes, the formed polynomials and the products with
several columns have to give the integers of a plain evaluation, to the last one."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

pytestmark = pytest.mark.gpu


def _rows(rng, rows, cols, mean, diag=False):
    """Sparse rows of random +-1, their lengths spread around the mean."""
    m = int(rows * mean)
    i, j = rng.integers(0, rows, m), rng.integers(0, cols, m)
    A = sp.coo_matrix((rng.choice([-1.0, 1.0], m), (i, j)), shape=(rows, cols)).tocsr()
    A.data = np.sign(A.data) + (A.data == 0)  # repeated places too: +-1
    if diag:
        A = A.tolil() if rows < 2000 else A
        A = sp.csr_matrix(A)
        A = A - sp.diags(A.diagonal()) + sp.identity(rows)
    A = sp.csr_matrix(A)
    A.eliminate_zeros()
    A.sort_indices()
    return A


def _triple(A):
    return A.indptr, A.indices, A.data


# F points, C points, mean entries a row of A_ff, A_fc, Z and the coarsest matrix, degree
CASES = [
    (33, 9, 1.5, 2.0, 1.5, 4.0, 2),
    (700, 300, 6.0, 3.0, 9.0, 40.0, 1),
    (4000, 3000, 1.6, 2.5, 3.0, 30.0, 2),
    (20000, 9000, 12.0, 4.0, 4.0, 40.0, 1),
    (270000, 70000, 1.4, 3.0, 2.8, 6.0, 2),
    (300000, 280000, 3.0, 2.0, 3.0, 3.0, 1),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-{c[1]}")
@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("order", [0, 1])
def test_v_cycle_of_integers_is_exact(case, prec, order):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import Solver
    nf, nc, mff, mfc, mz, ma, d = case
    rng = np.random.default_rng(nf)
    Aff, Afc = _rows(rng, nf, nf, mff, True), _rows(rng, nf, nc, mfc)
    Z, A1 = _rows(rng, nc, nf, mz), _rows(rng, nc, nc, ma, True)
    state = np.full(nf + nc, 2, np.int8)
    F = np.sort(rng.permutation(nf + nc)[:nf])
    state[F] = 1
    C = np.flatnonzero(state == 2)
    cmap = rng.integers(-1, nc, nf).astype(np.int32)
    alpha = np.array([1.0, -1.0, 1.0][:d + 1])
    roots = np.array([1.0, 1.0, 1.0])
    top = sp.identity(nf + nc, format="csr")
    kw = dict(precision=prec, outer=1, max_it=1, locality_order=order)
    s = Solver.from_hierarchy(
        [dict(state=state, a=_triple(top), ff=_triple(Aff), fc=_triple(Afc), z=_triple(Z), cmap=cmap, alpha=alpha),
         dict(a=_triple(A1), roots=roots)], **kw)
    B = rng.integers(-2, 3, (64, nf + nc)).astype(np.float64)

    def cycle(b, op=lambda M: M):
        sgn = -1.0 if op(-1.0) == -1.0 else 1.0  # with op = abs: the sums of magnitudes
        rf, rc = b[F], b[C]
        rc = rc + op(Z) @ rf
        w, ec = rc, 0.0 * rc
        for k in range(len(roots)):
            ec = ec + w
            if k + 1 < len(roots):
                w = w + sgn * (op(A1) @ w)
        W = np.where((cmap >= 0)[:, None], ec[np.maximum(cmap, 0)], 0.0)
        sv = rf + sgn * (op(Afc) @ ec + op(Aff) @ W)
        y = alpha[-1] * sv if sgn < 0 else sv
        for a in alpha[-2::-1]:
            y = op(Aff) @ y + (a if sgn < 0 else 1.0) * sv
        e = np.zeros_like(b)
        e[F], e[C] = W + y, ec
        return e
    want = cycle(B.T).T
    # every partial sum in any order is an integer that FP32 holds
    assert cycle(np.abs(B.T), abs).max() < 2 ** 24
    for nrhs in (1, 2, 5, 16, 64) if nf < 200000 else (1, 4):
        b = torch.from_numpy(B[:nrhs]).cuda()
        x = s.solve(b if nrhs > 1 else b[0])[0].cpu().numpy().reshape(nrhs, -1)
        assert np.array_equal(x, want[:nrhs]), nrhs
    s.close()
