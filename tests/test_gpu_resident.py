"""1x1 nodes whose filters stay in registers: the GEMM's bits (same products, same order) and the oracle's values, at the edges of
an instance's channels, shares of the positions that end inside a tile, several tiles a workgroup (the ring wraps), strides,
padding, zero siblings.  NGC_RESIDENT=1: every node that fits."""
import numpy as np
import pytest
import torch

import oracle
import paper_1801_08058_amd as ng
from oracle import Attrs
from gpu_util import Run, bound
from test_gpu_parity import _tensors

pytestmark = pytest.mark.gpu
BLK = ng.NGC_NCHW16C

CASES = [
    # n  c    h   w   k   r  s  sh sw dh dw pbh pbw pah paw
    Attrs(1, 16, 1, 1, 16, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0),        # one position, one channel block
    Attrs(2, 64, 5, 7, 64, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0),
    Attrs(3, 80, 9, 11, 80, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),       # odd sizes, siblings past the edges
    Attrs(1, 128, 8, 6, 144, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),
    Attrs(2, 144, 7, 9, 128, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),
    Attrs(1, 256, 13, 5, 512, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),     # the most filters of either direction
    Attrs(1, 512, 6, 10, 256, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),
    Attrs(2, 272, 5, 5, 48, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0),       # 32 steps, the last 15 dead; 64 channels
    Attrs(1, 496, 4, 9, 16, 1, 1, 1, 3, 1, 1, 0, 0, 0, 0),       # 32 steps, 32 channels; a stride in one axis
    Attrs(2, 48, 6, 7, 272, 1, 1, 2, 2, 1, 1, 1, 1, 0, 1),       # padding: positions outside the image
    Attrs(9, 32, 61, 59, 48, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0),      # 32391 positions: shares of 128, tiles of 256
    Attrs(5, 240, 63, 41, 304, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0),    # several tiles of 32, the ring wraps
    Attrs(7, 160, 101, 71, 112, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),   # as above with siblings
    Attrs(5, 64, 79, 81, 400, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),     # backwards (400 to 64 channels, and 64 to 400 below) the GEMM
    Attrs(5, 400, 79, 81, 64, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),
    Attrs(9, 64, 61, 83, 48, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),      # every instance with siblings, several tiles a workgroup: 4 steps, 64 channels
    Attrs(7, 128, 61, 83, 32, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),     # ... 128 channels
    Attrs(5, 256, 61, 83, 64, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),     # ... 256
    Attrs(7, 128, 61, 83, 112, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),    # 8 steps, 128
    Attrs(5, 240, 61, 83, 128, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),    # ... 256
    Attrs(4, 384, 61, 83, 128, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),    # ... 512
    Attrs(7, 96, 61, 83, 240, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),     # 16 steps, 128
    Attrs(5, 256, 61, 83, 256, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),    # ... 256
    Attrs(7, 112, 61, 83, 320, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),    # 32 steps, 128
    Attrs(5, 208, 61, 83, 512, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),    # ... 256
    Attrs(3, 320, 65, 63, 240, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0),
]


def siblings_fit(a):
    """The channel counts (k to c) that have an instance for strided backprop-data."""
    return a.c <= 256 if a.k <= 64 else a.c > 64 and (a.k <= 128 or a.c <= 256)


@pytest.mark.parametrize("case", range(len(CASES)))
def test_resident_filters(case, monkeypatch):
    a = CASES[case]
    print("case", a, flush=True)
    x, w, b, dy = _tensors(a, "bf16", 18000 + case)
    monkeypatch.setenv("NGC_FWD_FEW", "0")
    run, got = Run(a, "bf16", BLK, BLK, True), {}
    for force in ("0", "1"):
        monkeypatch.setenv("NGC_RESIDENT", force)
        y = run.fwd(x, w, bias=b, relu=True)
        tail = ":resident" if force == "1" else ""
        assert ng.ngc_conv_kernel(run.last_desc, ng.NGC_OP_FWD) == "gemm1x1_bf16" + tail
        got[force] = [run.last_raw]
        dx = run.bwd_data(dy, w)
        if a.pbh == 0 and a.sw != 3:                             # one class of pixels, 2 x 2 of them a position
            assert ng.ngc_conv_kernel(run.last_desc, ng.NGC_OP_BWD_DATA) == "gemm1x1_bf16" + (tail if a.sh == 1 or siblings_fit(a) else "")
        got[force].append(run.last_raw)
    assert all(torch.equal(p, q) for p, q in zip(got["0"], got["1"]))
    if a.n * a.h * a.w < 4000:
        assert oracle.max_normalised_error(y, oracle.conv_fwd(a, x, w, bias=b, relu=True)) <= bound("bf16", "act")
        assert oracle.max_normalised_error(dx, oracle.conv_bwd_data_gather(a, dy, w)) <= bound("bf16", "act")
    assert not np.isnan(y).any() and not np.isnan(dx).any()
