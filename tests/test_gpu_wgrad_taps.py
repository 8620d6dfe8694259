"""Several-taps-per-pass backprop-filters (blocked bf16, rank 2 and 3) against the oracle: every number of taps a pass
holds, every width of k and c a workgroup holds, one part and several, strides, dilation, stages of whole small images
and slices, taps that lie outside the tensor altogether."""
import pytest

import oracle
import paper_1801_08058_amd as ng
from oracle import Attrs, Attrs3
from gpu_util import Run, Run3, bound
from test_gpu_conv3d import _check3, _tensors3
from test_gpu_parity import _tensors

pytestmark = pytest.mark.gpu
BLK = ng.NGC_NCHW16C

CASES = [
    # n  c   h   w   k   r  s  sh sw dh dw pbh pbw pah paw
    Attrs(2, 48, 9, 13, 80, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1),       # partial tiles of k and c
    Attrs(3, 16, 21, 40, 16, 3, 3, 2, 2, 1, 1, 1, 1, 1, 1),      # stride 2, rows evened out over stages
    Attrs(9, 32, 5, 6, 48, 2, 2, 2, 2, 1, 1, 0, 0, 0, 0),        # four taps; several whole images a stage, a ragged last one
    Attrs(2, 32, 12, 18, 32, 5, 5, 1, 1, 1, 1, 2, 2, 2, 2),      # 25 taps in groups of nine, the last of seven
    Attrs(1, 16, 7, 60, 64, 1, 7, 1, 1, 1, 1, 0, 3, 0, 3),       # seven taps
    Attrs(2, 64, 30, 4, 16, 7, 1, 2, 1, 1, 1, 3, 0, 3, 0),       # seven taps along h, stride 2
    Attrs(2, 16, 10, 10, 16, 3, 3, 1, 1, 3, 2, 3, 2, 3, 2),      # dilation
    Attrs(1, 16, 4, 230, 16, 1, 2, 1, 1, 1, 1, 0, 0, 0, 0),      # rows too long for a stage: the per-tap kernel
    Attrs(1, 32, 1, 1, 32, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1),        # one pixel: eight of the taps see padding only
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("force", [None, 11001, 22003, 34001, 44009])
def test_wgrad_taps(case, force, monkeypatch):
    """force: 16-channel blocks of k, of c, parts (10000s, 1000s, rest; beyond what a shape has: its own choice)."""
    if force:
        monkeypatch.setenv("NGC_WGRAD_TAPS", str(force))
    a = CASES[case]
    x, w, b, dy = _tensors(a, "bf16", 13000 + case)
    run = Run(a, "bf16", BLK, BLK, True)
    dw = run.bwd_filters(x, dy)
    assert ng.ngc_conv_variant(run.last_desc, ng.NGC_OP_BWD_FILTERS) == "wgrad_gemm_bf16"
    assert oracle.max_normalised_error(dw, oracle.conv_bwd_filters(a, x, dy)) <= bound("bf16", "dw")


CASES3 = [
    #      n  c   d  h  w   k   t  r  s  s  s  s  d  d  d  padding below, above
    Attrs3(2, 32, 5, 6, 7, 48, 3, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1),       # several slices a stage
    Attrs3(1, 16, 9, 19, 20, 80, 3, 3, 3, 2, 2, 2, 1, 1, 1, 1, 1, 1, 1, 1, 1),     # stride 2
    Attrs3(3, 16, 1, 8, 9, 16, 3, 2, 2, 1, 1, 1, 1, 1, 1, 1, 0, 0, 1, 1, 1),       # one slice: two depth taps outside
    Attrs3(2, 32, 1, 6, 8, 16, 1, 2, 3, 3, 1, 1, 1, 1, 1, 0, 0, 1, 2, 0, 1),       # one slice each, padding behind only
]


@pytest.mark.parametrize("case", range(len(CASES3)))
@pytest.mark.parametrize("force", [None, 11001, 42003])
def test_wgrad_taps_rank3(case, force, monkeypatch):
    if force:
        monkeypatch.setenv("NGC_WGRAD_TAPS", str(force))
    a = CASES3[case]
    _check3(a, "bf16", BLK, BLK, False, 13100 + case, ("", "", "wgrad_gemm3"))


@pytest.mark.parametrize("force", [None, 11001, 21002])
def test_wgrad_taps_rank3_one_slice_in_front_of_x(force, monkeypatch):
    """One depth tap, one slice of x and of dy, and the padding in front takes the tap outside x: dw is zero."""
    if force:
        monkeypatch.setenv("NGC_WGRAD_TAPS", str(force))
    a = Attrs3(2, 16, 1, 7, 9, 32, 1, 3, 3, 2, 1, 1, 1, 1, 1, 1, 1, 1, 0, 1, 1)
    x, w, b, dy = _tensors3(a, "bf16", 13200)
    assert (oracle.conv3d_bwd_filters(a, x, dy) == 0).all()
    assert (Run3(a, "bf16", BLK, BLK, False).bwd_filters(x, dy) == 0).all()
