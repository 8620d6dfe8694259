"""Forward / backprop-data of the nodes off the blocked kernels with operands straight to registers, against the oracle: both
ways of sharing out the work, at the edges of tiles, steps and filter rows (rows at odd 2-byte offsets, an odd last element of
the filter tensor, a last step with one index), the largest window it takes and the first it does not."""
import pytest

import oracle
import paper_1801_08058_amd as ng
from oracle import Attrs
from gpu_util import Run, bound
from test_gpu_parity import _tensors

pytestmark = pytest.mark.gpu
NCHW, BLK = ng.NGC_NCHW, ng.NGC_NCHW16C

CASES = [
    # n  c   h   w   k   r  s  sh sw dh dw pbh pbw pah paw
    (Attrs(1, 1, 5, 5, 1, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0), "bf16", NCHW, NCHW),        # one element each
    (Attrs(3, 17, 7, 11, 33, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0), "bf16", NCHW, NCHW),     # odd rows, odd tensor, one index past a step
    (Attrs(2, 9, 9, 13, 35, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "bf16", NCHW, NCHW),      # 81 indices, 315 rows of them
    (Attrs(2, 9, 9, 13, 35, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "f32", NCHW, NCHW),
    (Attrs(2, 23, 10, 12, 24, 3, 3, 2, 2, 1, 1, 1, 1, 1, 1), "bf16", BLK, BLK),      # four residue classes, padding lanes
    (Attrs(2, 65, 9, 15, 31, 3, 2, 2, 3, 1, 2, 2, 0, 1, 3), "f32", NCHW, BLK),       # classes without taps
    (Attrs(1, 40, 12, 9, 40, 5, 6, 1, 1, 1, 1, 2, 3, 2, 2), "f32", NCHW, NCHW),      # 30 taps
    (Attrs(1, 3, 40, 9, 5, 31, 1, 1, 1, 1, 1, 15, 0, 15, 0), "f32", NCHW, NCHW),     # 31
    (Attrs(1, 3, 12, 9, 5, 4, 8, 1, 1, 1, 1, 2, 4, 1, 3), "f32", NCHW, NCHW),        # 32: the gather GEMM
    (Attrs(1, 700, 6, 7, 33, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "f32", NCHW, NCHW),      # 6300 indices: near the table's end forward
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("share", ["1", "2", None])
def test_stream(case, share, monkeypatch):
    if share:
        monkeypatch.setenv("NGC_STREAM", share)
    a, dtype, xl, yl = CASES[case]
    x, w, b, dy = _tensors(a, dtype, 16000 + case)
    run = Run(a, dtype, xl, yl, False)
    y = run.fwd(x, w, bias=b, relu=True)
    assert ng.ngc_conv_variant(run.last_desc, ng.NGC_OP_FWD) == "direct:gather"
    takes = "stream" if share and a.r * a.s <= 31 else "gather"
    if share or a.r * a.s > 31:
        assert [ng.ngc_conv_kernel(run.last_desc, op) for op in (ng.NGC_OP_FWD, ng.NGC_OP_BWD_DATA)] == ["direct:" + takes] * 2
    assert oracle.max_normalised_error(y, oracle.conv_fwd(a, x, w, bias=b, relu=True)) <= bound(dtype, "act")
    assert oracle.max_normalised_error(run.bwd_data(dy, w), oracle.conv_bwd_data_gather(a, dy, w)) <= bound(dtype, "act")
    assert oracle.max_normalised_error(run.bwd_data_relu(dy, w, x), oracle.conv_bwd_data_relu(a, dy, w, x)) <= bound(dtype, "act")
