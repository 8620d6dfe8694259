"""Several-taps-per-pass backprop-filters (blocked bf16, rank 2 and 3) against the oracle: every number of taps a pass
holds, every width of k and c a workgroup holds, one part and several (both reduce kernels, parts dealt to the XCDs),
strides, dilation, stages of whole small images and slices, taps that lie outside the tensor altogether."""
import pytest

import oracle
import paper_1801_08058_amd as ng
from oracle import Attrs, Attrs3
from gpu_util import Run, Run3, bound
from test_gpu_conv3d import _check3, _tensors3
from test_gpu_parity import _tensors

pytestmark = pytest.mark.gpu
BLK = ng.NGC_NCHW16C

# node, taps a pass holds, forced splits it admits: 16-channel blocks of k, of c, parts (10000s, 1000s, rest)
CASES = [
    # n  c   h   w   k   r  s  sh sw dh dw pbh pbw pah paw
    (Attrs(2, 48, 9, 13, 80, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), 9, (11001, 22001, 34001, 44001)),   # partial tiles of k and c
    (Attrs(3, 16, 21, 40, 16, 3, 3, 2, 2, 1, 1, 1, 1, 1, 1), 9, (11001, 11003, 11006)),         # stride 2, rows evened out over stages
    (Attrs(9, 32, 5, 6, 48, 2, 2, 2, 2, 1, 1, 0, 0, 0, 0), 4, (11001, 32001)),                  # several whole images a stage, a ragged last one
    (Attrs(2, 32, 12, 18, 32, 5, 5, 1, 1, 1, 1, 2, 2, 2, 2), 9, (11001, 22002, 21002)),         # 25 taps in groups of nine, the last of seven
    (Attrs(1, 16, 7, 60, 64, 1, 7, 1, 1, 1, 1, 0, 3, 0, 3), 7, (11001, 41002)),
    (Attrs(2, 64, 30, 4, 16, 7, 1, 2, 1, 1, 1, 3, 0, 3, 0), 7, (11001, 14001)),                 # seven taps along h, stride 2
    (Attrs(2, 16, 10, 10, 16, 3, 3, 1, 1, 3, 2, 3, 2, 3, 2), 9, (11001,)),                      # dilation
    (Attrs(1, 32, 1, 1, 32, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), 9, (11001, 22001)),                  # one pixel: eight of the taps see padding only
    (Attrs(2, 48, 11, 30, 32, 1, 2, 1, 1, 1, 1, 0, 0, 0, 1), 2, (11001, 22002)),
    (Attrs(2, 48, 11, 30, 48, 1, 3, 1, 1, 1, 1, 0, 1, 0, 1), 3, (11001, 32002, 24001)),
    (Attrs(2, 32, 16, 20, 64, 5, 1, 1, 1, 1, 1, 2, 0, 2, 0), 5, (11001, 42003)),
    (Attrs(12, 64, 40, 40, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), 9, (44003, 44009, 42016, 44024, 44070)),   # many stages
    (Attrs(6, 80, 30, 36, 48, 2, 3, 1, 1, 1, 1, 0, 1, 1, 1), 7, (34008, 22016)),                # six taps in a pass of seven
]


def _split(a, nt, force):
    """Bytes of the partials of a forced split (whole 256 bytes; one part needs none)."""
    nkb, ncq, parts = force // 10000, force // 1000 % 10, force % 1000
    groups = -(-a.r * a.s // nt) * getattr(a, "t", 1)
    tiles = -(-a.k // (16 * nkb)) * -(-a.c // (16 * ncq)) * groups
    return 256 if parts == 1 else parts * tiles * ncq * nkb * nt * 1024


@pytest.mark.parametrize("case,force", [(i, f) for i, (_, _, forces) in enumerate(CASES) for f in (None,) + forces])
def test_wgrad_taps(case, force, monkeypatch):
    a, nt, _ = CASES[case]
    monkeypatch.setenv("NGC_WGRAD_STRIP", "0")
    if force:
        monkeypatch.setenv("NGC_WGRAD_TAPS", str(force))
    x, w, b, dy = _tensors(a, "bf16", 13000 + case)
    run = Run(a, "bf16", BLK, BLK, True)
    dw = run.bwd_filters(x, dy)
    if force:
        assert ng.ngc_conv_variant(run.last_desc, ng.NGC_OP_BWD_FILTERS) == "wgrad_gemm_bf16:taps"
        assert ng.ngc_conv_workspace_bytes(run.last_desc, ng.NGC_OP_BWD_FILTERS) == _split(a, nt, force)
    assert oracle.max_normalised_error(dw, oracle.conv_bwd_filters(a, x, dy)) <= bound("bf16", "dw")


def test_rows_too_long_for_a_stage_stay_with_the_per_tap_kernel():
    a = Attrs(1, 16, 4, 230, 16, 1, 2, 1, 1, 1, 1, 0, 0, 0, 0)
    x, w, b, dy = _tensors(a, "bf16", 13050)
    run = Run(a, "bf16", BLK, BLK, True)
    dw = run.bwd_filters(x, dy)
    assert ng.ngc_conv_variant(run.last_desc, ng.NGC_OP_BWD_FILTERS) == "wgrad_gemm_bf16"
    assert oracle.max_normalised_error(dw, oracle.conv_bwd_filters(a, x, dy)) <= bound("bf16", "dw")


# the all-taps strip kernel's nodes that are handed over: few positions, which leave its fixed split idle
@pytest.mark.parametrize("a", [Attrs(1, 64, 14, 14, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), Attrs(4, 128, 7, 7, 128, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1)])
def test_strip_kernel_hands_small_nodes_over(a):
    x, w, b, dy = _tensors(a, "bf16", 13060 + a.n)
    run = Run(a, "bf16", BLK, BLK, True)
    dw = run.bwd_filters(x, dy)
    assert ng.ngc_conv_variant(run.last_desc, ng.NGC_OP_BWD_FILTERS) == "wgrad_strip_bf16:taps"
    assert oracle.max_normalised_error(dw, oracle.conv_bwd_filters(a, x, dy)) <= bound("bf16", "dw")


CASES3 = [
    #      n  c   d  h  w   k   t  r  s  s  s  s  d  d  d  padding below, above
    (Attrs3(2, 32, 5, 6, 7, 48, 3, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1), 9, (11001, 22002)),      # several slices a stage
    (Attrs3(1, 16, 9, 19, 20, 80, 3, 3, 3, 2, 2, 2, 1, 1, 1, 1, 1, 1, 1, 1, 1), 9, (11001, 41003)),    # stride 2
    (Attrs3(3, 16, 1, 8, 9, 16, 3, 2, 2, 1, 1, 1, 1, 1, 1, 1, 0, 0, 1, 1, 1), 4, (11001,)),            # one slice: two depth taps outside
    (Attrs3(2, 32, 1, 6, 8, 16, 1, 2, 3, 3, 1, 1, 1, 1, 1, 0, 0, 1, 2, 0, 1), 7, (11001,)),            # one slice each, padding behind only
    (Attrs3(2, 48, 7, 9, 12, 64, 3, 1, 1, 1, 2, 2, 1, 1, 1, 1, 0, 0, 1, 0, 0), 1, (11001, 42002, 44001)),   # one tap a pass
    # many parts: no multiple of 8 and a multiple (then the tiles of a part on one XCD), 64 and more of any count
    (Attrs3(6, 32, 12, 16, 20, 48, 3, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1), 9, (11009, 21013, 22016, 12065)),
]


@pytest.mark.parametrize("case,force", [(i, f) for i, (_, _, forces) in enumerate(CASES3) for f in (None,) + forces])
def test_wgrad_taps_rank3(case, force, monkeypatch):
    a, nt, _ = CASES3[case]
    if force:
        monkeypatch.setenv("NGC_WGRAD_TAPS", str(force))
        d = ng.make_desc3(a.n, a.c, a.d, a.h, a.w, a.k, a.t, a.r, a.s, (a.sd, a.sh, a.sw), (a.dd, a.dh, a.dw), (a.pbd, a.pbh, a.pbw), (a.pad, a.pah, a.paw))
        assert ng.ngc_conv3d_workspace_bytes(d, ng.NGC_OP_BWD_FILTERS) == _split(a, nt, force)
    _check3(a, "bf16", BLK, BLK, False, 13100 + case, ("", "", "wgrad_gemm3_bf16:taps" if force else "wgrad_gemm3"))


@pytest.mark.parametrize("force", [None, 11001, 21002])
def test_wgrad_taps_rank3_one_slice_in_front_of_x(force, monkeypatch):
    """One depth tap, one slice of x and of dy, and the padding in front takes the tap outside x: dw is zero."""
    if force:
        monkeypatch.setenv("NGC_WGRAD_TAPS", str(force))
    a = Attrs3(2, 16, 1, 7, 9, 32, 1, 3, 3, 2, 1, 1, 1, 1, 1, 1, 1, 1, 0, 1, 1)
    x, w, b, dy = _tensors3(a, "bf16", 13200)
    assert (oracle.conv3d_bwd_filters(a, x, dy) == 0).all()
    assert (Run3(a, "bf16", BLK, BLK, False).bwd_filters(x, dy) == 0).all()
