"""Convolutions of any channel count: on the register-staged kernel (fp32 data
and channel counts that are no multiple of 8) at the edges of its runs (one
filter row of s * c elements, padded to 8 16-bit or 4 fp32 ones), tiles and K
steps, and on the direct-to-LDS kernel for multiples of 8; all three passes
against the oracle; NaN around every operand must not reach a result."""
import numpy as np
import pytest

import workloads as W
from oracle import ops
from oracle.rounding import decode
from tests.helpers import DT, accum_bound, dev, host64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mdnn():
    import torch
    torch.cuda.set_device(0)
    import paper_2011_11188_amd as m
    return m


# (n, h, w, c_in, c_out, r, s, pad): three channels with wide filters (runs of
# 21, 15, 9), a run one over and one under a chunk, channels either side of 64
# and 128, one-pixel-wide images, valid and over-wide padding, r != s, a
# tall output (128 x 64 tiles backward, gathered forward), split filter gradients with a ragged last step.
SHAPES = [
    (2, 11, 9, 3, 64, 7, 7, 3), (3, 8, 8, 3, 70, 5, 5, 2), (2, 6, 7, 3, 130, 3, 3, 1), (5, 13, 11, 17, 33, 3, 3, 1),
    (2, 7, 5, 65, 67, 3, 3, 0), (1, 9, 1, 20, 129, 3, 3, 1), (2, 5, 6, 12, 9, 1, 1, 0), (2, 4, 5, 100, 12, 1, 5, 2),
    (3, 6, 6, 10, 11, 2, 4, 3), (2, 180, 190, 7, 60, 3, 3, 1), (4, 30, 31, 5, 13, 3, 3, 1),
    # 128 x 128 tiles in both directions (518 of them forward, also enough for
    # fp32); 128 x 64 forward with a reduction too long to be gathered
    (2, 182, 184, 70, 70, 1, 3, 0), (2, 182, 184, 70, 60, 1, 3, 0),
    # 2^22 outputs backward, either side of the shortest reduction's rule
    (2, 128, 129, 128, 4, 1, 1, 0), (2, 128, 129, 128, 5, 1, 1, 0),
]


@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_conv_any_channels(mdnn, shape, dt):
    _check(mdnn, shape, dt, 1)


# Channel counts that are multiples of 8 but not of 64, on the direct-to-LDS
# kernel: one chunk per tap, a K step over several taps and filter rows, K and
# pixel counts that end inside a step, valid and over-wide padding (filter
# gradients whose output grid is not the input's), outputs that take the 256 x
# 64 tile past 128 columns (200), the 128 x 64 and the 64 x 128 one, one-pixel-wide images.
SHAPES8 = [
    (2, 9, 7, 8, 16, 3, 3, 1), (3, 8, 8, 24, 40, 5, 5, 2), (2, 7, 9, 72, 88, 3, 3, 0), (1, 6, 5, 16, 8, 3, 3, 2),
    (4, 13, 1, 40, 136, 3, 3, 1), (2, 10, 11, 48, 200, 1, 1, 0), (9, 11, 13, 96, 80, 5, 5, 2), (2, 5, 6, 104, 72, 2, 4, 3),
    (3, 90, 91, 8, 200, 3, 3, 1), (5, 12, 13, 64, 64, 3, 3, 0), (2, 6, 6, 8, 8, 7, 7, 3),
    # narrow outputs of 66248 and 66976 pixels: 256 x 64 tiles, not 128 x 64, by
    # the 64-channel loaders one way and the runs of 40 channels the other
    (2, 182, 184, 64, 40, 1, 3, 0), (2, 182, 184, 40, 64, 1, 3, 0),
]


@pytest.mark.parametrize("dt", ["f16", "bf16"])
@pytest.mark.parametrize("shape", SHAPES8)
def test_conv_multiples_of_8_channels(mdnn, shape, dt):
    _check(mdnn, shape, dt, 8)


# Images or filters of less than one 16-byte chunk: read by elements, steps of
# several filter rows, output channels past 16 and past the filter's chunk.
TINY = [(1, 1, 1, 1, 1, 1, 1, 0), (7, 1, 1, 1, 2, 3, 3, 1), (3, 1, 1, 2, 9, 3, 3, 1), (1, 2, 2, 1, 40, 2, 2, 1),
        (9, 5, 7, 3, 2, 1, 1, 0), (300, 4, 3, 7, 1, 1, 1, 0), (2, 1, 1, 3, 33, 5, 5, 4), (4, 9, 1, 1, 1, 7, 1, 0),
        (1, 1, 1, 3, 300, 1, 1, 0)]


@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("shape", TINY)
def test_conv_below_a_chunk(mdnn, shape, dt):
    _check(mdnn, shape, dt, 1)


def _check(mdnn, shape, dt, gap):
    """All three passes, each operand `gap` elements into a buffer of NaN."""
    import torch
    n, h, w, ci, co, r, s, pad = shape
    ho, wo = h + 2 * pad - r + 1, w + 2 * pad - s + 1
    arr = {"x": W.normal((n, h, w, ci), 61, 1, dt), "w": W.normal((co, r, s, ci), 61, 2, dt),
           "dy": W.normal((n, ho, wo, co), 61, 3, dt)}
    val = {k: decode(v, dt) for k, v in arr.items()}
    mag = {k: np.abs(v) for k, v in val.items()}
    buf, t = {}, {}
    for k, v in arr.items():
        d = dev(v, dt).reshape(-1)
        buf[k] = torch.full((d.numel() + 2 * gap,), float("nan"), dtype=d.dtype, device="cuda")
        t[k] = buf[k][gap:-gap]
        t[k].copy_(d)
    sh = mdnn.ConvShape(n, h, w, ci, co, r, s, pad)
    y = torch.full((n, ho, wo, co), float("nan"), device="cuda")
    dx = torch.full((n, h, w, ci), float("nan"), device="cuda")
    dw, db = torch.full((co, r, s, ci), float("nan"), device="cuda"), torch.empty(co, device="cuda")
    ws = torch.full((max(mdnn.mdnn_conv2d_bwd_filter_workspace(sh, DT[dt]), 256),), 255, dtype=torch.uint8, device="cuda")
    mdnn.mdnn_conv2d_fwd(sh, t["x"], t["w"], DT[dt], None, 0, y, DT["f32"])
    mdnn.mdnn_conv2d_bwd_data(sh, t["dy"], t["w"], DT[dt], None, dx, DT["f32"])
    mdnn.mdnn_conv2d_bwd_filter(sh, t["x"], t["dy"], DT[dt], dw, db, ws, ws.numel())
    for name, got, want, size, k in (
            ("y", y, ops.conv2d_fwd(val["x"], val["w"], pad), ops.conv2d_fwd(mag["x"], mag["w"], pad), r * s * ci),
            ("dx", dx, ops.conv2d_bwd_data(val["dy"], val["w"], pad, h, w),
             ops.conv2d_bwd_data(mag["dy"], mag["w"], pad, h, w), r * s * co),
            ("dw", dw, ops.conv2d_bwd_filter(val["x"], val["dy"], pad, r, s),
             ops.conv2d_bwd_filter(mag["x"], mag["dy"], pad, r, s), n * ho * wo),
            ("db", db, val["dy"].sum((0, 1, 2)), mag["dy"].sum((0, 1, 2)), n * ho * wo)):
        err = np.abs(host64(got) - want)
        assert np.all(err <= accum_bound(size, k + 1)), (name, shape, dt, float(np.nanmax(err)), bool(np.isnan(err).any()))


def test_conv_tall_image_reads_nothing_past_the_filter(mdnn):
    """An image of more than 2^24 rows: the K steps end in rows past the
    filter, which must stay outside the image for every output (an Inf four
    rows below an output, one row past the filter, must not reach it)."""
    import torch
    h, ci, r, pad, row = (1 << 24) + 4096, 5, 7, 3, 10
    x = torch.zeros((1, h, 1, ci), dtype=torch.float16, device="cuda")
    x[0, row] = float("inf")
    wt = torch.ones((1, r, r, ci), dtype=torch.float16, device="cuda")
    y = torch.full((1, h, 1, 1), float("nan"), device="cuda")
    mdnn.mdnn_conv2d_fwd(mdnn.ConvShape(1, h, 1, ci, 1, r, r, pad), x, wt, DT["f16"], None, 0, y, DT["f32"])
    want = torch.zeros_like(y)
    want[0, row - pad:row + pad + 1] = float("inf")
    assert torch.equal(y, want)
