"""Products on the register-staged kernel: operands whose rows start on any
element (odd leading dimensions, offset bases, any K) and fp32 operands, at
the edges of its tiles, chunks and K steps, against the fp64 definition.
Bar: fp32 accumulation of K exact (16-bit) or once-rounded (fp32) products,
gamma_{K+1} * sum |a b| (helpers.accum_bound), elementwise."""
import numpy as np
import pytest

import workloads as W
from oracle import ops
from oracle.rounding import decode
from tests.helpers import DT, accum_bound, dev, host64, lowp_close

pytestmark = pytest.mark.gpu
LAYOUT = {"NN": 0, "NT": 1, "TN": 2}


@pytest.fixture(scope="module")
def mdnn():
    import torch
    torch.cuda.set_device(0)
    import paper_2011_11188_amd as m
    return m


# (M, N, K): either side of a chunk (8 / 4 elements), a K step (64 / 32), of
# the 64- and 128-wide tiles; 2050 x 2049: 128 x 128 tiles; K of one element
# past a step; the smallest extents the kernel takes.
SHAPES = [(9, 8, 9), (65, 63, 64), (64, 64, 65), (127, 129, 31), (130, 66, 33), (33, 257, 321), (200, 72, 129),
          (2050, 2049, 70)]

# Few K steps and many outputs, either side of the rules that pick a kernel or
# tile for them: 2^17, 2^18, 2^20 and 2^21 outputs, K of 16, 48 and 128, 384 tiles
# of 128 x 128.
SHALLOW = [(361, 364, 16), (513, 516, 5), (510, 513, 9), (700, 375, 128), (701, 375, 129), (1023, 1028, 16),
           (1023, 1028, 17), (1449, 1452, 48), (1449, 1452, 49), (2433, 2561, 65), (2432, 2560, 128)]


@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("layout", ["NN", "NT", "TN"])
def test_register_staged_any_alignment(mdnn, layout, dt):
    _check(mdnn, layout, dt, SHAPES)


@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("layout", ["NN", "NT", "TN"])
def test_register_staged_few_steps(mdnn, layout, dt):
    _check(mdnn, layout, dt, SHALLOW)


def _check(mdnn, layout, dt, shapes):
    import torch
    for i, (m, n, k) in enumerate(shapes):
        sa = (k, m) if layout == "TN" else (m, k)
        sb = (n, k) if layout == "NT" else (k, n)
        a = W.normal(sa, 51, 10 * i + 1, dt)
        b = W.normal(sb, 51, 10 * i + 2, dt)
        want = ops.gemm(layout, decode(a, dt), decode(b, dt))
        bound = accum_bound(ops.gemm(layout, np.abs(decode(a, dt)), np.abs(decode(b, dt))), k + 1)
        # bases off by one and three elements, odd leading dimensions; NaN
        # around the operands must not reach the result
        def place(x, skip, pad):
            t = dev(x, dt)
            buf = torch.full((skip + x.shape[0] * (x.shape[1] + pad),), float("nan"), dtype=t.dtype, device="cuda")
            v = buf[skip:].view(x.shape[0], x.shape[1] + pad)
            v[:, :x.shape[1]] = t
            return buf, v
        for skip, pad in ((0, 0), (1, 3), (3, 1)):
            ka, A = place(a, skip, pad)
            kb, B = place(b, skip, pad)
            D = torch.full((m, n), float("nan"), dtype=torch.float32, device="cuda")
            mdnn.mdnn_gemm_mixed(LAYOUT[layout], m, n, k, 1.0, A, A.stride(0), B, B.stride(0), DT[dt], 0.0, None, 0, D,
                                 n, DT["f32"])
            got = host64(D)
            assert np.all(np.abs(got - want) <= bound), (layout, dt, (m, n, k), skip, pad,
                                                         float(np.max(np.abs(got - want) - bound)))


@pytest.mark.parametrize("dt", ["f16", "bf16"])
def test_register_staged_epilogue_and_split(mdnn, dt):
    """Bias, ReLU, mask and beta * C stored in the storage type and in fp32 with
    odd row strides, and K split over a workspace (the last split ragged)."""
    import torch
    for m, n, k in ((131, 77, 1001), (40, 70, 2000)):
        a, b = W.normal((m, k), 52, 1, dt, 1 / np.sqrt(k)), W.normal((k, n), 52, 2, dt)
        bias, mk = W.normal((n,), 52, 3, "f32", 0.5), W.normal((m, n), 52, 4, dt)
        D = torch.zeros((m, n + 1), dtype=dev(a, dt).dtype, device="cuda")
        flag = torch.zeros(1, dtype=torch.int32, device="cuda")
        mdnn.gemm(mdnn.NN, dev(a, dt), dev(b, dt), bias=dev(bias, "f32"), act=1, mask=dev(mk, dt), out=D[:, :n],
                  workspace=True, nonfinite=flag)
        a64, b64 = decode(a, dt), decode(b, dt)
        exact = np.where(decode(mk, dt) > 0, ops.bias_act(ops.gemm("NN", a64, b64), bias.astype(np.float64), "relu"), 0)
        assert lowp_close(host64(D)[:, :n], exact, dt, accum_bound(np.abs(a64) @ np.abs(b64) + np.abs(bias), k + 1))
        assert not host64(D)[:, n].any() and flag.item() == 0
        # the kernel's own epilogue (no split), alpha and beta * C added, both output types
        for odt in (dt, "f32"):
            c = W.normal((m, n + 3), 52, 5, odt)
            D = torch.zeros((m, n + 1), dtype=dev(c, odt).dtype, device="cuda")
            mdnn.gemm(mdnn.NN, dev(a, dt), dev(b, dt), bias=dev(bias, "f32"), act=1, mask=dev(mk, dt), out=D[:, :n],
                      alpha=0.5, beta=-2.0, Cm=dev(c, odt)[:, :n], nonfinite=flag)
            c64 = decode(c, odt)[:, :n]
            z = 0.5 * ops.gemm("NN", a64, b64) - 2.0 * c64 + bias
            exact = np.where(decode(mk, dt) > 0, np.maximum(z, 0.0), 0.0)
            bound = accum_bound(np.abs(a64) @ np.abs(b64) + 2 * np.abs(c64) + np.abs(bias), k + 3)
            got = host64(D)
            if odt == "f32":
                assert np.all(np.abs(got[:, :n] - exact) <= bound)
            else:
                assert lowp_close(got[:, :n], exact, dt, bound)
            assert not got[:, n].any() and flag.item() == 0
