"""Backprop-filters of NCHW tensors off the blocked kernels with operands straight to registers, against the oracle: one part and
several, at the edges of tiles, units and rows (odd 2-byte offsets, units that start in front of the tensor, an odd
last element); without a workspace; infinities where taps lie in the padding or a unit ends past its row."""
import numpy as np
import pytest
import torch

import oracle
import paper_1801_08058_amd as ng
from oracle import Attrs
from gpu_util import Run, bound, data_to_device, desc_of, stream
from test_gpu_parity import _tensors

pytestmark = pytest.mark.gpu
NCHW = ng.NGC_NCHW

CASES = [
    # n  c   h   w   k   r  s  sh sw dh dw pbh pbw pah paw
    (Attrs(1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0), "bf16"),            # one position
    (Attrs(3, 7, 13, 11, 33, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "f32"),          # one k past a tile, 63 columns
    (Attrs(3, 7, 13, 11, 33, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "bf16"),         # odd rows
    (Attrs(2, 15, 9, 8, 70, 5, 5, 1, 1, 1, 1, 2, 2, 2, 2), "bf16"),          # whole units, two in front of the tensor
    (Attrs(5, 41, 11, 13, 97, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0), "bf16"),        # an image as one row, odd tensors
    (Attrs(5, 41, 12, 13, 97, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0), "f32"),
    (Attrs(2, 6, 17, 19, 20, 5, 4, 2, 3, 2, 1, 1, 4, 3, 0), "f32"),          # strides, dilation, one-sided padding
    (Attrs(2, 9, 17, 19, 20, 3, 3, 2, 2, 1, 1, 1, 1, 1, 1), "bf16"),
    (Attrs(1, 3, 9, 5, 8, 3, 9, 1, 1, 1, 1, 1, 8, 1, 8), "f32"),             # more padding than a unit
    (Attrs(1, 3, 9, 5, 8, 3, 9, 2, 1, 1, 1, 1, 8, 1, 8), "bf16"),
    (Attrs(1, 2, 6, 300, 5, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "f32"),           # long rows
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("parts", [None, 1, 2, 7])
def test_wgrad_stream(case, parts, monkeypatch):
    a, dtype = CASES[case]
    if parts:
        monkeypatch.setenv("NGC_WGRAD_STREAM", str(parts))
    x, w, b, dy = _tensors(a, dtype, 17000 + case)
    run = Run(a, dtype, NCHW, NCHW, False)
    dw = run.bwd_filters(x, dy)
    if parts:
        assert ng.ngc_conv_kernel(run.last_desc, ng.NGC_OP_BWD_FILTERS) == "direct:stream"
    assert oracle.max_normalised_error(dw, oracle.conv_bwd_filters(a, x, dy)) <= bound(dtype, "dw")


def test_without_workspace():
    a = CASES[1][0]
    x, w, b, dy = _tensors(a, "f32", 17100)
    d = desc_of(a, "f32", NCHW, NCHW)
    dw = torch.full((a.k * a.c * a.r * a.s,), float("nan"), device="cuda")
    ng.ngc_conv_bwd_filters(d, data_to_device(x, "f32", NCHW), data_to_device(dy, "f32", NCHW), dw, None, stream())
    torch.cuda.synchronize()
    got = dw.cpu().numpy().astype(np.float64).reshape(a.k, a.c, a.r, a.s)
    assert oracle.max_normalised_error(got, oracle.conv_bwd_filters(a, x, dy)) <= bound("f32", "dw")


@pytest.mark.parametrize("parts", [1, 4])
def test_zeros_in_place_of_positions_meet_infinities(parts, monkeypatch):
    """An infinite x under the end of a row, an infinite dy whose taps lie in the padding: sums without them stay finite."""
    monkeypatch.setenv("NGC_WGRAD_STREAM", str(parts))
    a = Attrs(2, 5, 6, 7, 34, 3, 3, 1, 1, 1, 1, 0, 0, 1, 1)                  # 5 x 6 positions: two of a row's second unit are none
    x, w, b, dy = _tensors(a, "f32", 17200)
    x[1, 2, 3, 6], dy[0, 7, 4, 5] = np.inf, np.inf
    got = Run(a, "f32", NCHW, NCHW, False).bwd_filters(x, dy)
    with np.errstate(invalid="ignore"):
        xp = np.pad(x.astype(np.float64), ((0, 0), (0, 0), (0, 1), (0, 1)))
        want = np.zeros((a.k, a.c, 3, 3))
        for r in range(3):
            for s in range(3):
                rows, cols = min(5, a.h - r), min(6, a.w - s)
                want[:, :, r, s] = np.einsum("nkpq,ncpq->kc", dy[:, :, :rows, :cols].astype(np.float64), xp[:, :, r:r + rows, s:s + cols])
    assert np.array_equal(np.isfinite(got), np.isfinite(want)) and np.array_equal(np.isnan(got), np.isnan(want))
    f = np.isfinite(want)
    assert np.abs(got[f] - want[f]).max() <= 1e-5 * np.abs(want[f]).max()
