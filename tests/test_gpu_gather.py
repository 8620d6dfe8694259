"""Gather GEMM kernels (fp32 tensors, channel counts off the block, first layers) against the oracle: every tile of
forward / backprop-data and of backprop-filters, one part and several, at sizes around the edges of their tiles and
steps; the split reduction without a workspace."""
import pytest
import torch

import oracle
import paper_1801_08058_amd as ng
from oracle import Attrs
from gpu_util import Run, bound, data_to_device, desc_of, stream
from test_gpu_parity import _check_all, _tensors

pytestmark = pytest.mark.gpu
NCHW, BLK = ng.NGC_NCHW, ng.NGC_NCHW16C

CASES = [
    # n  c   h   w   k   r  s  sh sw dh dw pbh pbw pah paw
    (Attrs(1, 1, 5, 5, 1, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0), "f32", NCHW, NCHW),         # one output channel, one index
    (Attrs(3, 7, 13, 11, 33, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "f32", NCHW, NCHW),      # one channel past a tile
    (Attrs(2, 16, 8, 16, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "f32", NCHW, NCHW),      # whole tiles, aligned filter rows
    (Attrs(2, 65, 9, 15, 31, 3, 2, 2, 3, 1, 2, 2, 0, 1, 3), "f32", NCHW, BLK),       # strides and dilation: classes without taps
    (Attrs(1, 5, 40, 37, 66, 5, 5, 4, 3, 1, 1, 2, 2, 2, 2), "f32", BLK, NCHW),       # largest stride the classes hold
    (Attrs(2, 3, 33, 35, 40, 7, 7, 2, 2, 1, 1, 3, 3, 3, 3), "bf16", NCHW, BLK),      # first layer, width off the 16-byte grid
    (Attrs(4, 40, 14, 14, 72, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "bf16", NCHW, NCHW),
    (Attrs(1, 3, 40, 9, 5, 31, 1, 1, 1, 1, 1, 15, 0, 15, 0), "f32", NCHW, NCHW),     # longest window
    (Attrs(1, 3, 40, 9, 5, 32, 1, 1, 1, 1, 1, 15, 0, 15, 0), "f32", NCHW, NCHW),     # one tap more: the one-thread-per-output kernels
    (Attrs(1, 2, 12, 12, 3, 3, 3, 5, 1, 1, 1, 1, 1, 1, 1), "bf16", NCHW, NCHW),      # one stride more
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("tile,wgrad", [(None, None), (1, 1001), (2, 2001), (3, 3001), (1, 1003), (2, 2002), (3, 3005)])
def test_gather_tiles(case, tile, wgrad, monkeypatch):
    a, dtype, xl, yl = CASES[case]
    if tile:
        monkeypatch.setenv("NGC_GATHER_TILE", str(tile))
        monkeypatch.setenv("NGC_GATHER_WGRAD", str(wgrad))
    names = ["direct:gather"] * 3
    if a.r > 31:
        names = ["direct"] * 3
    elif max(a.sh, a.sw) > 4:
        names[1] = "direct"
    _check_all(a, dtype, xl, yl, False, 12000 + case, names)
    assert ng.ngc_conv_variant(desc_of(a, dtype, xl, yl), ng.NGC_OP_FWD) == names[0]


def test_backprop_filters_without_a_workspace():
    """The partial sums' workspace is optional for these nodes: without it one part runs, same result to fp32 rounding."""
    a = Attrs(6, 20, 24, 24, 24, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1)
    x, w, b, dy = _tensors(a, "f32", 12100)
    d = desc_of(a, "f32", NCHW, NCHW)
    assert ng.ngc_conv_workspace_bytes(d, ng.NGC_OP_BWD_FILTERS) > 0
    dw = torch.full((a.k * a.c * 9,), float("nan"), dtype=torch.float32, device="cuda")
    ng.ngc_conv_bwd_filters(d, data_to_device(x, "f32", NCHW), data_to_device(dy, "f32", NCHW), dw, None, stream())
    torch.cuda.synchronize()
    got = dw.cpu().numpy().astype("float64").reshape(a.k, a.c, 3, 3)
    assert oracle.max_normalised_error(got, oracle.conv_bwd_filters(a, x, dy)) <= bound("f32", "dw")
    assert oracle.max_normalised_error(Run(a, "f32", NCHW, NCHW, False).bwd_filters(x, dy), got) <= bound("f32", "dw")
