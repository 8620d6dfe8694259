"""Multi-tap nodes whose waves split the reduction, against the oracle: tiles of whole images and of rows, a second tile that does not
exist, images past the batch, channel counts that end inside a tile or a 32-channel chunk, chunks of fewer steps than a chunk has
blocks to load, patches of exactly the largest size, strides, dilations.  NGC_WAVES=1: every node that fits."""
import numpy as np
import pytest

import oracle
import paper_1801_08058_amd as ng
from oracle import Attrs
from gpu_util import Run, bound
from test_gpu_parity import _check_backward_compounds, _tensors

pytestmark = pytest.mark.gpu
BLK = ng.NGC_NCHW16C

CASES = [
    # n  c    h   w   k   r  s  sh sw dh dw pbh pbw pah paw
    Attrs(5, 64, 7, 7, 80, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1),        # two images a tile, the last tile one; channels end in the second tile
    Attrs(2, 48, 14, 14, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1),      # rows of an image; an odd 16-channel block
    Attrs(1, 32, 5, 6, 16, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1),        # one tile: the other waves have none; 9 steps, unequal quarters
    Attrs(3, 128, 9, 11, 32, 1, 2, 1, 1, 1, 1, 0, 0, 0, 1),      # two taps: chunks shorter than their loads
    Attrs(3, 272, 6, 8, 48, 2, 1, 1, 1, 1, 1, 1, 0, 0, 0),       # as above, nine chunks, the last half empty
    Attrs(2, 96, 23, 10, 64, 5, 5, 1, 1, 1, 1, 2, 2, 2, 2),      # 25 taps, a last strip of fewer rows
    Attrs(2, 128, 1, 140, 32, 1, 3, 1, 2, 1, 1, 0, 1, 0, 1),   # one row, stride 2: 141 patch pixels
    Attrs(2, 64, 1, 112, 32, 1, 5, 1, 1, 1, 2, 0, 4, 0, 4),      # 112 positions a row, dilated taps
    Attrs(4, 160, 12, 13, 112, 2, 2, 2, 2, 1, 1, 0, 0, 0, 0),    # stride 2 without padding (backwards: four classes, the strip kernel)
    Attrs(3, 64, 13, 9, 64, 3, 3, 1, 1, 2, 2, 2, 2, 2, 2),       # dilation
    Attrs(2, 64, 10, 9, 64, 3, 3, 1, 1, 1, 1, 0, 2, 2, 0),       # the halo on one side only
    Attrs(2, 64, 12, 9, 64, 3, 3, 1, 1, 1, 1, 0, 0, 0, 0),       # no padding; full correlation backwards
    Attrs(7, 512, 4, 4, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1),       # several images a tile, 36 steps a wave
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("pre", [True, False])
def test_waves(case, pre, monkeypatch):
    a = CASES[case]
    print("case", a, flush=True)
    x, w, b, dy = _tensors(a, "bf16", 19000 + case)
    monkeypatch.setenv("NGC_FWD_FEW", "0")
    monkeypatch.setenv("NGC_WAVES", "1")
    run = Run(a, "bf16", BLK, BLK, pre)
    for bias, relu in ((b, True), (None, False)):
        y = run.fwd(x, w, bias=bias, relu=relu)
        assert ng.ngc_conv_kernel(run.last_desc, ng.NGC_OP_FWD) == "strip_bf16:waves"
        assert oracle.max_normalised_error(y, oracle.conv_fwd(a, x, w, bias=bias, relu=relu)) <= bound("bf16", "act")
    dx = run.bwd_data(dy, w)
    assert (ng.ngc_conv_kernel(run.last_desc, ng.NGC_OP_BWD_DATA) == "strip_bf16:waves") == (a.sh == a.sw == 1 and (a.k + 31) // 32 * a.r * a.s >= 8)
    ref = oracle.conv_bwd_data_gather(a, dy, w)
    assert oracle.max_normalised_error(dx, ref) <= bound("bf16", "act")
    _check_backward_compounds(run, a, x, w, dy, ref, bound("bf16", "act"))


def test_waves_special_values(monkeypatch):
    """Infinities and NaN reach the positions that the strip kernel gives them, and no others."""
    a = CASES[0]
    x, w, b, dy = _tensors(a, "bf16", 19100)
    x[1, 17, 3, 2], x[4, 40, 0, 6], dy[0, 5, 6, 6], dy[3, 70, 2, 0] = np.inf, np.nan, -np.inf, np.nan
    monkeypatch.setenv("NGC_FWD_FEW", "0")
    run, got = Run(a, "bf16", BLK, BLK, True), {}
    for force in ("0", "1"):
        monkeypatch.setenv("NGC_WAVES", force)
        got[force] = run.fwd(x, w, bias=b), run.bwd_data(dy, w)
        assert ng.ngc_conv_kernel(run.last_desc, ng.NGC_OP_BWD_DATA).endswith(":waves") == (force == "1")
    for p, q in zip(got["0"], got["1"]):
        assert np.isnan(p).any() and np.isinf(p).any()
        assert np.array_equal(np.isnan(p), np.isnan(q)) and np.array_equal(np.isinf(p), np.isinf(q))
        ok = np.isfinite(p)
        assert np.abs(p[ok] - q[ok]).max() <= 2 * bound("bf16", "act") * np.abs(p[ok]).max()
