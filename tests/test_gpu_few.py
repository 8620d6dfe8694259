"""Forward of nodes with few output tiles (blocked bf16, rank 2) against the oracle: ragged tiles of channels and positions,
both numbers of waves, fewer units of the reduction than waves and more than a batch, strides, dilation, one-sided
padding, windows that reach outside the image."""
import pytest

import oracle
import paper_1801_08058_amd as ng
from oracle import Attrs
from gpu_util import Run, bound
from test_gpu_parity import _tensors

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
