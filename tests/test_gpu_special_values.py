"""Infinities at places the sums must not reach: elements of the padding, of channels and of positions past the end."""
import numpy as np
import pytest

import oracle
import paper_1801_08058_amd as ng
from oracle import Attrs
from gpu_util import Run, bound, host
from test_gpu_parity import _tensors

pytestmark = pytest.mark.gpu
NCHW, BLK = ng.NGC_NCHW, ng.NGC_NCHW16C

# the kernels of these nodes: tiles of the gather GEMM, operands straight to registers with either share of the work, the default
TILES = [1, 2, 3, "positions", "slices", None]


def _force(monkeypatch, tile, wgrad=None):
    if tile in ("positions", "slices"):
        monkeypatch.setenv("NGC_STREAM", "1" if tile == "positions" else "2")
    elif tile:
        monkeypatch.setenv("NGC_GATHER_TILE", str(tile))
    if wgrad and wgrad < 1000:
        monkeypatch.setenv("NGC_WGRAD_STREAM", str(wgrad))
    elif wgrad:
        monkeypatch.setenv("NGC_GATHER_WGRAD", str(wgrad))


def _runs(run, op, tile):
    name = ng.ngc_conv_kernel(run.last_desc, op)
    assert name in ("direct:stream", "direct:gather") if tile is None else name == ("direct:stream" if isinstance(tile, str) else "direct:gather")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tile", TILES)
def test_infinite_filter_leaves_the_padding_lanes_zero(dtype, tile, monkeypatch):
    """Reduction indices past the end meet output channels past the end: both read zero, not filter element 0."""
    _force(monkeypatch, tile)
    a = Attrs(1, 5, 6, 6, 20, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1)
    x, w, b, dy = _tensors(a, dtype, 15000)
    w[0, 0, 0, 0] = np.inf
    run = Run(a, dtype, BLK, BLK, False)
    bits = np.uint16 if dtype == "bf16" else np.uint32
    y = run.fwd(x, w, bias=b, relu=False)
    _runs(run, ng.NGC_OP_FWD, tile)
    assert np.all(host(run.last_raw, bits).reshape(1, 2, 6, 6, 16)[:, 1, :, :, 4:] == 0)
    w0 = w.copy()
    w0[0] = 0
    assert oracle.max_normalised_error(y[:, 1:], oracle.conv_fwd(a, x, w0, bias=b)[:, 1:]) <= bound(dtype, "act")
    run.bwd_data(dy, w)
    _runs(run, ng.NGC_OP_BWD_DATA, tile)
    assert np.all(host(run.last_raw, bits).reshape(1, 1, 6, 6, 16)[..., 5:] == 0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tile", TILES)
def test_infinite_input_leaves_the_padding_lanes_zero(dtype, tile, monkeypatch):
    _force(monkeypatch, tile)
    a = Attrs(1, 5, 6, 6, 20, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1)
    x, w, b, dy = _tensors(a, dtype, 15001)
    x[0, 2, 3, 3] = np.inf
    dy[0, 7, 2, 2] = -np.inf
    run = Run(a, dtype, BLK, BLK, False)
    bits = np.uint16 if dtype == "bf16" else np.uint32
    run.fwd(x, w, bias=b, relu=False)
    assert np.all(host(run.last_raw, bits).reshape(1, 2, 6, 6, 16)[:, 1, :, :, 4:] == 0)
    run.bwd_data(dy, w)
    _runs(run, ng.NGC_OP_BWD_DATA, tile)
    assert np.all(host(run.last_raw, bits).reshape(1, 1, 6, 6, 16)[..., 5:] == 0)


def _same(got, ref, tol):
    """Finite where the oracle is, within tol of its largest finite value; the same infinities and NaNs elsewhere."""
    fin = np.isfinite(ref)
    assert fin.any()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    assert np.abs(got[fin] - ref[fin]).max() / np.abs(ref[fin]).max() <= tol


PADDED = [
    # n  c   h   w   k   r  s  sh sw dh dw pbh pbw pah paw
    (Attrs(2, 7, 9, 11, 33, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "f32", NCHW, NCHW),
    (Attrs(2, 20, 8, 8, 21, 3, 2, 2, 3, 1, 2, 2, 0, 1, 3), "f32", NCHW, BLK),
    (Attrs(1, 5, 12, 10, 17, 5, 5, 2, 1, 1, 1, 2, 2, 2, 2), "bf16", BLK, NCHW),
    (Attrs(3, 9, 8, 8, 40, 3, 3, 1, 1, 2, 2, 2, 2, 2, 2), "bf16", NCHW, NCHW),
    (Attrs(2, 12, 6, 6, 12, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1), "f32", NCHW, NCHW),       # one tap, a frame of padding only
    (Attrs(2, 9, 11, 13, 37, 3, 3, 2, 2, 1, 1, 1, 1, 1, 1), "bf16", NCHW, NCHW),     # strided columns
    (Attrs(2, 7, 9, 10, 34, 5, 5, 1, 1, 1, 1, 2, 2, 2, 2), "bf16", NCHW, NCHW),      # units two elements in front of the tensor
    (Attrs(1, 5, 9, 5, 8, 3, 9, 1, 1, 1, 1, 1, 8, 1, 8), "f32", NCHW, NCHW),         # more padding than a unit
    (Attrs(1, 11, 7, 9, 40, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "bf16", BLK, BLK),
]


@pytest.mark.parametrize("case", range(len(PADDED)))
@pytest.mark.parametrize("tile,wgrad", [(1, 1001), (2, 2001), (3, 3003), ("positions", 1), ("slices", 3), (None, None)])
def test_infinities_meet_no_padding(case, tile, wgrad, monkeypatch):
    """A tap in the padding is no part of the sum: an infinite filter element or gradient does not turn it into NaN."""
    _force(monkeypatch, tile, wgrad)
    a, dtype, xl, yl = PADDED[case]
    x, w, b, dy = _tensors(a, dtype, 15100 + case)
    run = Run(a, dtype, xl, yl, False)
    wi = w.copy()
    wi[a.k // 2, a.c // 2, 0, 0] = np.inf
    wi[2, 1, a.r - 1, a.s - 1] = -np.inf
    _same(run.fwd(x, wi, bias=b), oracle.conv_fwd(a, x, wi, bias=b), bound(dtype, "act"))
    _runs(run, ng.NGC_OP_FWD, tile)
    _same(run.bwd_data(dy, wi), oracle.conv_bwd_data_gather(a, dy, wi), bound(dtype, "act"))
    _runs(run, ng.NGC_OP_BWD_DATA, tile)
    di = dy.copy()
    di[0, a.k // 2, 0, 0] = np.inf
    di[a.n - 1, 1, -1, -1] = np.nan
    _same(run.bwd_filters(x, di), oracle.conv_bwd_filters(a, x, di), bound(dtype, "dw"))
    _runs(run, ng.NGC_OP_BWD_FILTERS, tile if xl == yl == NCHW else 1 if tile else None)   # blocked tensors: the gather GEMM


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tile", TILES)
def test_infinities_of_the_next_filter_row(dtype, tile, monkeypatch):
    """Filter rows of 63 elements, no multiple of a step: an infinity or NaN at the start of a row is no part of the row before."""
    _force(monkeypatch, tile)
    a = Attrs(2, 7, 6, 9, 35, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1)
    x, w, b, dy = _tensors(a, dtype, 15150)
    w[1::4, 0, 0, 0] = np.inf
    w[3::4, 0, 0, 1] = np.nan
    for xl, yl in ((NCHW, NCHW), (BLK, NCHW)):
        run = Run(a, dtype, xl, yl, False)
        got, ref = run.fwd(x, w, bias=b), oracle.conv_fwd(a, x, w, bias=b)
        _runs(run, ng.NGC_OP_FWD, tile)
        _same(got, ref, bound(dtype, "act"))
        assert np.isfinite(got[:, 0::2]).all()


TAPS = [
    # n  c   h   w   k   r  s  sh sw dh dw pbh pbw pah paw
    (Attrs(1, 32, 9, 11, 32, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), [(8, 10)]),                # one stage, 99 positions
    (Attrs(3, 16, 7, 7, 48, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), [(6, 6), (0, 0)]),           # whole images, 49 positions each
    (Attrs(2, 32, 21, 60, 32, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), [(20, 0), (20, 59)]),      # a last block of fewer rows
    (Attrs(2, 16, 24, 50, 64, 2, 2, 2, 2, 1, 1, 0, 0, 0, 0), [(23, 49), (23, 0)]),
    (Attrs(1, 64, 13, 29, 16, 5, 5, 1, 1, 1, 1, 2, 2, 2, 2), [(12, 3), (11, 28)]),
]


@pytest.mark.parametrize("case", range(len(TAPS)))
@pytest.mark.parametrize("force", [None, 11001, 21002, 11003])
def test_infinite_inputs_meet_no_position_past_the_end(case, force, monkeypatch):
    """Backprop-filters of several taps per pass: positions are multiplied 32 at a time, those past the last one of a stage
    are no part of the sum, whatever x holds where their taps would reach."""
    if force:
        monkeypatch.setenv("NGC_WGRAD_TAPS", str(force))
    a, pixels = TAPS[case]
    x, w, b, dy = _tensors(a, "bf16", 15200 + case)
    dy[dy == 0] = 0.5                                     # zero times infinity is the oracle's to find, not here
    for i, (h, ww) in enumerate(pixels):
        x[a.n - 1, 1 + i, h, ww] = (-1) ** i * np.inf
    run = Run(a, "bf16", BLK, BLK, False)
    _same(run.bwd_filters(x, dy), oracle.conv_bwd_filters(a, x, dy), bound("bf16", "dw"))
