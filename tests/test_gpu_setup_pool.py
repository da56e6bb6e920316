"""The blocks a setup keeps while it runs: setups on several threads and streams
at once, failing setups between them, and memory given back."""
import ctypes
import threading

import numpy as np
import pytest
import torch

from airg_inputs import workloads

pytestmark = pytest.mark.gpu


def _in_use(lib):
    v = ctypes.c_int64()
    assert lib.airg_set_alloc_budget(0, ctypes.byref(v)) == 0
    return v.value


def test_setups_on_threads_and_streams_keep_their_results_and_give_memory_back():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_17517_amd import AirgError, Solver, binding
    lib = binding.load()
    probs = [workloads.fv_random(n, 0.5, True, seed=60 + n) for n in (70, 33, 120)]
    before = _in_use(lib)

    def one(p, stream):
        with torch.cuda.stream(stream):
            with pytest.raises(AirgError):  # a zero diagonal ends this setup early
                bad = p.data.copy()
                bad[p.indices == np.repeat(np.arange(p.n), np.diff(p.indptr))] = 0.0
                Solver(p.indptr, p.indices, bad)
            s = Solver(p.indptr, p.indices, p.data)
            b = torch.from_numpy(p.b).cuda()
            x, i = s.solve(b)
            lam, _ = s.adjoint_solve(b)  # a second setup in the same handle
            s.close()
            assert i["converged"] == 1
            return x.cpu().numpy(), lam.cpu().numpy()

    alone = [one(p, torch.cuda.current_stream()) for p in probs]
    got = {}

    def work(k):
        got[k] = [one(p, s) for p, s in [(probs[k], torch.cuda.Stream()) for _ in range(3)]]

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(probs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k, (x, lam) in enumerate(alone):
        assert len(got[k]) == 3
        for y, mu in got[k]:
            assert np.array_equal(x, y) and np.array_equal(lam, mu)
    assert _in_use(lib) == before
