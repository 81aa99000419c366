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


class _Geom(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("n", "h", "w", "c", "k", "r", "s", "pad", "ho", "wo")]


class _Plan(C.Structure):
    _fields_ = [("splits", C.c_int), ("k_per_split", C.c_int64)]


def _geom(n, h, w, c, k, r, pad):
    return _Geom(n, h, w, c, k, r, r, pad, h + 2 * pad - r + 1, w + 2 * pad - r + 1)


def test_direct_to_lds_filter_gradient_offsets_fit_32_bits(lib):
    """Few pixels and very many output channels: dy's byte offsets up to the end
    of the padded last K step (64 pixels) stay below 2^32, where the range check
    turns them into zeros (past it they would wrap to valid rows, and an Inf
    there would reach the sums as 0 * Inf)."""
    f = lib["_ZN4mdnn21conv_pipe_filter_planERKNS_8ConvGeomE"]
    f.argtypes, f.restype = [C.POINTER(_Geom)], _Plan
    taken = 0
    for n in (1, 2, 3, 15, 16, 31, 32, 33, 63, 64, 65, 129):
        for k in [8, 64, 1 << 20] + [(1 << p) + d for p in (24, 25, 26) for d in (-8, 0, 8)]:
            if f(C.byref(_geom(n, 1, 1, 8, k, 1, 0))).splits:
                taken += 1
                assert -(-n // 64) * 64 * k * 2 <= 2 ** 32, (n, k)
    assert taken > 40


def test_direct_to_lds_convolution_launches_stay_below_2_32_threads(lib):
    """More output pixels than 512 threads per 128 x 128 or 256 x 64 tile leave
    room for go to the general kernel, whose launch still holds them."""
    fit = lib["_ZN4mdnn18conv_pipe_runs_fitEll"]
    fit.argtypes, fit.restype = [C.c_int64, C.c_int64], C.c_bool
    taken = 0
    for n in (1, 64, 65, 72, 128, 129, 1000):
        for m in [64, 1 << 20] + [(1 << p) + d for p in (27, 28, 29, 30, 31) for d in (-300, -1, 0)]:
            if fit(m, n):
                taken += 1
                assert 512 * max(-(-m // 128) * -(-n // 128), -(-m // 256) * -(-n // 64)) < 2 ** 32, (m, n)
    assert taken > 30 and all(fit(1 << 20, n) for n in (1, 64, 200, 1000))
