"""CPU checks of the rules that choose a kernel, through the library's own
functions (no GPU work)."""
import ctypes as C

import pytest


@pytest.fixture(scope="module")
def lib():
    import paper_2011_11188_amd as m
    return C.CDLL(m.LIB_PATH)


def test_column_sums_one_launch_rule(lib):
    """One launch of 1024-thread blocks: only above one 256-row chunk (below,
    most of its row lanes would have no row) and within a launch's 2^32 threads."""
    f = lib["_ZN4mdnn16column_sums_onceEll"]
    f.argtypes, f.restype = [C.c_int64, C.c_int64], C.c_bool
    for cols in (8, 64, 1000, 1 << 20):
        assert not any(f(rows, cols) for rows in (0, 1, 32, 255, 256, 1025, 5000))
        assert all(f(rows, cols) for rows in (257, 1000, 1024))
    assert not f(1024, 7)
    for cols in ((1 << 28) - 64, (1 << 28) - 63, 1 << 28, (1 << 28) + 70, 1 << 40):
        assert not f(300, cols) or -(-cols // 64) * 1024 < 2 ** 32
