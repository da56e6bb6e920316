"""Arithmetic on the positions of a matrix's entries next to the limit of 2^31 - 1
entries that the setup accepts (host builds of what the kernels use)."""
import ctypes

import numpy as np
import pytest

from paper_2508_17517_amd import binding

LAST = 2 ** 31 - 1


@pytest.mark.parametrize("s,e", [(0, 5), (LAST - 1, LAST), (LAST - 63, LAST), (LAST - 2048, LAST),
                                 (LAST - 5000, LAST), (LAST - 5000, LAST - 1), (LAST, LAST)])
def test_walks_end_at_the_row_s_end(s, e):
    host = binding.load_host_dense()
    out = (ctypes.c_uint32 * 20000)()
    for chunk in (1, 1024, 2048):  # entry-staged, row-block and setup products
        n = host.airg_host_walk_entries(s, e, chunk, 0, 10000, out)
        assert n == -(-(e - s) // chunk)
        got = [x for k in range(n) for x in range(out[2 * k], out[2 * k + 1])]
        assert got == list(range(s, e))
    for stride in (4, 64, 256):  # a group of lanes a row
        got = []
        for lane in range(min(stride, 64)):
            n = host.airg_host_walk_entries(s, e, -stride, lane, 10000, out)
            assert n <= 10000
            got += [out[2 * k] for k in range(n)]
        lanes = min(stride, 64)
        assert sorted(got) == [p for p in range(s, e) if (p - s) % stride < lanes]


@pytest.mark.parametrize("hi", [100, 2 ** 30 + 50, 2 ** 30 + 100, LAST])
def test_searches_far_into_a_matrix(hi):
    host = binding.load_host_dense()
    # positions hi - 100 .. hi - 1 of a column array that would be 8 GB whole
    col = np.arange(0, 300, 3, dtype=np.int32)
    at = col.ctypes.data - 4 * (hi - 100)
    for k, c in enumerate(col):
        assert host.airg_host_find_col(at, hi - 100, hi, int(c)) == hi - 100 + k
        assert host.airg_host_find_col(at, hi - 100, hi, int(c) + 1) == -1
        assert host.airg_host_first_from(at, hi - 100, hi, int(c)) == hi - 100 + k
        assert host.airg_host_first_from(at, hi - 100, hi, int(c) + 1) == hi - 99 + k


def test_pairs_of_entries():
    host = binding.load_host_dense()
    for e in (0, 1, 2, 7, LAST - 1, LAST):
        assert host.airg_host_pairs_before(e) == (e + 1) // 2
