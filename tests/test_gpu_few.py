"""Forward and backprop-data of nodes with few output tiles (blocked bf16) against the oracle: ragged tiles of channels and
positions, both numbers of waves, both tiles, fewer units of the reduction than waves and more than a batch, strides, dilation,
one-sided padding, windows that reach outside the image, classes of dx that no tap reaches, three spatial axes.  The staged
kernels, which these nodes keep with the switch off, are run on them as well."""
import pytest

import oracle
import paper_1801_08058_amd as ng
from oracle import Attrs, Attrs3
from gpu_util import Run, bound, desc3_of
from test_gpu_conv3d import _check3
from test_gpu_parity import _check_backward_compounds, _tensors

pytestmark = pytest.mark.gpu
BLK = ng.NGC_NCHW16C

CASES = [
    # n  c    h   w   k   r  s  sh sw dh dw pbh pbw pah paw
    Attrs(1, 16, 1, 1, 16, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0),        # one unit, one position, half a channel tile
    Attrs(2, 48, 5, 7, 48, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0),        # two images in a tile
    Attrs(1, 1024, 14, 14, 32, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0),    # 64 units: eight waves, whole batches
    Attrs(1, 1040, 3, 11, 80, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0),     # 65: sixteen waves
    Attrs(1, 256, 7, 7, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1),       # 144 units: two batches
    Attrs(3, 32, 9, 10, 48, 3, 3, 2, 1, 1, 2, 0, 2, 1, 2),       # stride, dilation, one-sided padding
    Attrs(1, 16, 6, 33, 112, 1, 7, 1, 2, 1, 1, 0, 3, 0, 3),
    Attrs(2, 16, 4, 4, 16, 5, 5, 1, 1, 1, 1, 4, 4, 4, 4),        # more padding than image
    Attrs(2, 32, 8, 8, 32, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),        # strided 1x1
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("epilogue", [False, True])
@pytest.mark.parametrize("force", ["1", None])
def test_few_tiles_forward(case, epilogue, force, monkeypatch):
    if force:
        monkeypatch.setenv("NGC_FWD_FEW", force)
    a = CASES[case]
    x, w, b, dy = _tensors(a, "bf16", 14000 + case)
    bias = b if epilogue else None
    run = Run(a, "bf16", BLK, BLK, True)
    y = run.fwd(x, w, bias=bias, relu=epilogue)
    if force:
        assert ng.ngc_conv_variant(run.last_desc, ng.NGC_OP_FWD).endswith("_bf16:few")
    ref = oracle.conv_fwd(a, x, w, bias=bias, relu=epilogue)
    assert oracle.max_normalised_error(y, ref) <= bound("bf16", "act")


BWD_CASES = CASES + [
    Attrs(2, 32, 9, 8, 48, 2, 2, 3, 3, 1, 1, 0, 0, 0, 0),        # classes no tap reaches, pixels past the last window
    Attrs(1, 48, 7, 9, 32, 3, 3, 2, 2, 2, 2, 2, 2, 2, 2),        # stride and dilation share a factor: all taps in one class
    Attrs(1, 32, 1, 5, 32, 1, 3, 4, 2, 1, 3, 0, 3, 0, 3),        # fewer rows than classes
    Attrs(3, 80, 6, 7, 112, 5, 5, 1, 1, 1, 1, 2, 2, 2, 2),
]


@pytest.mark.parametrize("case", range(len(BWD_CASES)))
@pytest.mark.parametrize("pre", [False, True])
@pytest.mark.parametrize("force", ["1", "2", "0", None])
def test_few_tiles_backward(case, pre, force, monkeypatch):
    if force:
        monkeypatch.setenv("NGC_FWD_FEW", force)
    a = BWD_CASES[case]
    x, w, b, dy = _tensors(a, "bf16", 14100 + case)
    run = Run(a, "bf16", BLK, BLK, pre)
    dx = run.bwd_data(dy, w)
    if force:
        assert ng.ngc_conv_kernel(run.last_desc, ng.NGC_OP_BWD_DATA).endswith(":few") == (force != "0")
    ref = oracle.conv_bwd_data(a, dy, w)
    assert oracle.max_normalised_error(dx, ref) <= bound("bf16", "act")
    _check_backward_compounds(run, a, x, w, dy, ref, bound("bf16", "act"))
    if force == "2":                                             # the larger tile, forward
        y = run.fwd(x, w, bias=b, relu=True)
        assert oracle.max_normalised_error(y, oracle.conv_fwd(a, x, w, bias=b, relu=True)) <= bound("bf16", "act")


CASES3 = [
    # n  c    d  h  w   k   t  r  s  strides    dilation   pad below  pad above
    Attrs3(1, 16, 3, 3, 3, 16, 3, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1),
    Attrs3(2, 48, 4, 5, 7, 80, 3, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1),     # ragged tiles, two images in one
    Attrs3(1, 32, 5, 6, 9, 112, 3, 3, 3, 2, 2, 2, 1, 1, 1, 1, 1, 1, 1, 1, 1),    # eight classes
    Attrs3(2, 32, 7, 5, 6, 32, 2, 2, 2, 3, 2, 2, 1, 1, 1, 0, 0, 0, 0, 0, 0),     # classes no tap reaches
    Attrs3(1, 32, 4, 6, 5, 48, 3, 1, 3, 1, 2, 1, 2, 1, 1, 2, 0, 0, 0, 1, 2),
]


@pytest.mark.parametrize("case", range(len(CASES3)))
@pytest.mark.parametrize("force", ["1", "2", "0", None])
def test_few_tiles_three_axes(case, force, monkeypatch):
    if force:
        monkeypatch.setenv("NGC_FWD_FEW", force)
    if force:
        d = desc3_of(CASES3[case], "bf16", BLK, BLK)
        for op in (ng.NGC_OP_FWD, ng.NGC_OP_BWD_DATA):
            assert ng.ngc_conv3d_kernel(d, op) == ("strip3_bf16" if force == "0" else "strip3_bf16:few")
    _check3(CASES3[case], "bf16", BLK, BLK, case % 2 == 0, 14300 + case, ("strip3_bf16", "strip3_bf16", "wgrad_gemm3"))
