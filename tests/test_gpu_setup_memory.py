"""Memory of the setup: what the library says it holds covers what the allocator
handed out, with and without a budget."""
import ctypes

import pytest
import torch

from airg_inputs import workloads

pytestmark = pytest.mark.gpu

NOMEM = -5
USED_CURRENT = 7  # hipMemPoolAttrUsedMemCurrent


def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


class _DevicePool:
    """Bytes that the device's stream-ordered allocator has handed out."""

    def __init__(self):
        self.hip = ctypes.CDLL("libamdhip64.so")
        self.pool = ctypes.c_void_p()
        assert self.hip.hipDeviceGetDefaultMemPool(ctypes.byref(self.pool), 0) == 0

    def used(self):
        v = ctypes.c_uint64()
        assert self.hip.hipMemPoolGetAttribute(self.pool, USED_CURRENT, ctypes.byref(v)) == 0
        return v.value


def _budget(lib, nbytes):
    held = ctypes.c_int64()
    assert lib.airg_set_alloc_budget(nbytes, ctypes.byref(held)) == 0
    return held.value


def test_bytes_held_and_the_budget_cover_what_is_allocated():
    _needs_gpu()
    from paper_2508_17517_amd import AirgError, Solver, binding
    lib = binding.load()
    pool = _DevicePool()
    p = workloads.fv_random(256, 0.3, True)  # 2^16 points: vectors of powers of two
    torch.cuda.synchronize()
    base, used0 = _budget(lib, 0), pool.used()
    assert used0 <= base
    s = Solver(p.indptr, p.indices, p.data)
    torch.cuda.synchronize()
    held = _budget(lib, 0) - base
    # every block of the allocator is one buffer and its 256 spare bytes
    assert pool.used() - used0 <= held
    s.close()
    torch.cuda.synchronize()
    assert _budget(lib, 0) == base and pool.used() == used0
    done = 0
    try:
        for f in (0.5, 0.8, 1.0, 1.1, 1.25, 1.5, 2.0, 3.0):
            limit = base + int(f * held)
            _budget(lib, limit)
            try:
                s = Solver(p.indptr, p.indices, p.data)
                done += 1
                torch.cuda.synchronize()
                assert pool.used() <= limit, f
                s.close()
            except AirgError as e:
                assert e.code == NOMEM
            torch.cuda.synchronize()
            assert _budget(lib, 0) == base and pool.used() == used0
    finally:
        _budget(lib, 0)
    assert 0 < done < 8
