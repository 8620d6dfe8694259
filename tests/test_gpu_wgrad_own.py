"""Backprop-filters of 3x3-class windows whose waves take stages of their own, against the oracle: stages of a full step and of less,
a last row block of fewer rows, patches of every number of blocks, fewer stages than waves, one part and several (both reduce kernels,
parts dealt to the XCDs), strides, dilation.  NGC_WGRAD_TAPS = 41000 + parts asks for the tile that has such stages."""
import numpy as np
import pytest

import oracle
import paper_1801_08058_amd as ng
from oracle import Attrs
from gpu_util import Run, bound
from test_gpu_parity import _tensors

pytestmark = pytest.mark.gpu
BLK = ng.NGC_NCHW16C

CASES = [
    # n  c   h   w   k   r  s  sh sw dh dw pbh pbw pah paw      parts
    (Attrs(5, 48, 7, 7, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), (1, 2, 8)),           # 28 and 21 positions; 10 stages
    (Attrs(1, 16, 1, 5, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), (1,)),                # one stage: seven waves have none; one row
    (Attrs(3, 16, 8, 16, 128, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), (1, 3)),            # 32 positions, every step full; patch of 72
    (Attrs(2, 32, 9, 32, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), (1, 16)),            # rows of 32; patch of four blocks
    (Attrs(2, 16, 23, 28, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), (1, 9, 24)),        # a row a stage, three blocks
    (Attrs(2, 32, 13, 14, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), (1, 4)),            # two rows a stage, the last one row
    (Attrs(3, 16, 11, 13, 64, 3, 3, 2, 2, 1, 1, 1, 1, 1, 1), (1, 2)),            # stride 2
    (Attrs(3, 16, 9, 9, 64, 3, 3, 1, 1, 2, 2, 2, 2, 2, 2), (1, 2)),              # dilation
    (Attrs(4, 16, 6, 6, 64, 3, 3, 1, 1, 1, 1, 0, 0, 0, 0), (1,)),                # no padding: 16 positions, whole images
    (Attrs(2, 16, 3, 21, 64, 1, 9, 1, 1, 1, 1, 0, 4, 0, 4), (1, 2)),             # nine taps in a row
    (Attrs(6, 32, 7, 7, 80, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), (1, 3)),              # a tile of k with one 16-channel block
    (Attrs(3, 16, 10, 12, 112, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), (1, 2, 15)),       # ... with three; a stage a part
    (Attrs(40, 32, 7, 7, 192, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), (1, 5)),            # the rings go round
]


@pytest.mark.parametrize("case,parts", [(i, p) for i, (_, ps) in enumerate(CASES) for p in ps])
def test_own_stages(case, parts, monkeypatch):
    a = CASES[case][0]
    print("case", a, parts, flush=True)
    monkeypatch.setenv("NGC_WGRAD_STRIP", "0")
    monkeypatch.setenv("NGC_WGRAD_TAPS", str(41000 + parts))
    x, w, b, dy = _tensors(a, "bf16", 20000 + case)
    run = Run(a, "bf16", BLK, BLK, True)
    dw = run.bwd_filters(x, dy)
    assert ng.ngc_conv_variant(run.last_desc, ng.NGC_OP_BWD_FILTERS) == "wgrad_gemm_bf16:taps"
    assert ng.ngc_conv_kernel(run.last_desc, ng.NGC_OP_BWD_FILTERS) == "wgrad_gemm_bf16:taps_own"
    assert oracle.max_normalised_error(dw, oracle.conv_bwd_filters(a, x, dy)) <= bound("bf16", "dw")


def test_own_stages_special_values(monkeypatch):
    """Infinities and NaN reach the elements of dw that they reach through common stages, and no others: positions past the end of a
    stage, pixels past the patch and stages past the last one hold or meet zeros."""
    a = CASES[0][0]
    x, w, b, dy = _tensors(a, "bf16", 20100)
    x[0, 3, 4, 0], x[4, 17, 6, 6], x[2, 40, 0, 0], dy[1, 9, 3, 6] = np.inf, np.nan, -np.inf, np.inf
    monkeypatch.setenv("NGC_WGRAD_STRIP", "0")
    monkeypatch.setenv("NGC_WGRAD_TAPS", "41001")
    run = Run(a, "bf16", BLK, BLK, True)
    own = run.bwd_filters(x, dy)
    assert ng.ngc_conv_kernel(run.last_desc, ng.NGC_OP_BWD_FILTERS) == "wgrad_gemm_bf16:taps_own"
    monkeypatch.setenv("NGC_WGRAD_OWN", "0")
    common = run.bwd_filters(x, dy)
    assert ng.ngc_conv_kernel(run.last_desc, ng.NGC_OP_BWD_FILTERS) == "wgrad_gemm_bf16:taps"
    assert np.isnan(common).any() and np.isfinite(common).any()
    assert np.array_equal(np.isnan(own), np.isnan(common)) and np.array_equal(np.isinf(own), np.isinf(common))


@pytest.mark.parametrize("n,c,h,w,k,stride", [(16, 64, 9, 9, 256, 1), (8, 256, 14, 14, 64, 1), (32, 256, 9, 9, 512, 2), (16, 128, 28, 28, 80, 1)])
def test_own_stages_without_the_switches(n, c, h, w, k, stride):
    """The plan and the parts that the dispatcher chooses by itself: 3, 4, 1 and 8 parts."""
    a = Attrs(n, c, h, w, k, 3, 3, stride, stride, 1, 1, 1, 1, 1, 1)
    x, wt, b, dy = _tensors(a, "bf16", 20200 + c)
    run = Run(a, "bf16", BLK, BLK, True)
    dw = run.bwd_filters(x, dy)
    assert ng.ngc_conv_kernel(run.last_desc, ng.NGC_OP_BWD_FILTERS).endswith(":taps_own")
    assert oracle.max_normalised_error(dw, oracle.conv_bwd_filters(a, x, dy)) <= bound("bf16", "dw")
