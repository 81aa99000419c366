"""CPU checks of the register-staged kernels' addresses: the loaders' own
arithmetic, compiled for the host, against the operands' extents, over the
products and layers that the host's rules admit."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("host") / "host_loaders.so")
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
                    os.path.join(ROOT, "tests", "host_loaders.hip"), "-o", so], check=True, capture_output=True)
    return C.CDLL(so)


@pytest.fixture(scope="module")
def lib():
    import paper_2011_11188_amd as m
    return C.CDLL(m.LIB_PATH)


def _gemm_reg_ok(lib):
    f = lib["_ZN4mdnn11gemm_reg_okE12mdnn_dtype_t13mdnn_layout_tllllli"]
    f.argtypes, f.restype = [C.c_int, C.c_int] + [C.c_int64] * 5 + [C.c_int], C.c_bool
    return f


@pytest.mark.parametrize("dt,es", [(0, 4), (1, 2)])
def test_k_contiguous_chunks_stay_inside_the_operand(host, lib, dt, es):
    """K-contiguous operands of just under 4 GiB, K below and above a K step:
    whatever the rule admits is fetched from inside the operand (offsets are
    32-bit, and a K step's last chunks lie past a shorter K)."""
    ok, outside = _gemm_reg_ok(lib), host.host_mat_last_outside
    outside.argtypes, outside.restype = [C.c_int] + [C.c_int64] * 3, C.c_int64
    e, bk, lim = 16 // es, 128 // es, 2 ** 32 // es
    admitted = 0
    for k in sorted({e, e + 1, 2 * e, bk // 2 - 1, bk // 2, bk - e, bk - 1, bk, bk + 1, 3 * bk - 3}):
        for ld in sorted({k, k + 1, 2 * bk, 1000}):
            if ld < k:
                continue
            most = (lim - 1 - k) // ld + 1  # rows of the largest operand below 2^32 bytes
            for rows in (most, most - 1, most - bk // ld - 1, 65, 1000):
                for layout in (0, 1):  # NN: A alone is K-contiguous; NT: B too
                    if ok(dt, layout, rows, 64, k, ld, 64 if layout == 0 else k, 1):
                        admitted += 1
                        assert outside(dt, rows, ld, k) == 0, (k, ld, rows, layout)
                if ok(dt, 1, 64, rows, k, k, ld, 1):
                    assert outside(dt, rows, ld, k) == 0, (k, ld, rows, "B")
    assert admitted > 100


@pytest.mark.parametrize("dt", [0, 1])
@pytest.mark.parametrize("shape", [(2, 11, 9, 3, 64, 7, 3), (2, 6, 7, 3, 130, 3, 1), (5, 13, 11, 17, 33, 3, 1),
                                   (2, 7, 5, 65, 67, 3, 0), (1, 9, 1, 20, 129, 3, 1), (2, 5, 6, 12, 9, 1, 0)])
def test_run_chunks_are_shifted_by_less_than_a_chunk(host, shape, dt):
    """Chunks that lie wholly outside an image or filter are not kept, and must
    not be shifted either: a shift of a whole chunk or more is undefined."""
    f = host.host_conv_bad_shifts
    f.restype = C.c_int64
    assert f(dt, *shape) == 0
