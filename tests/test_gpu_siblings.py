"""Backprop-data of strided 1x1 nodes against the oracle: the stores that write a computed pixel's three zero siblings with it
pass a wave's results through LDS, 16 positions a store.  Odd image sizes (siblings outside the image), position counts that end
inside a wave's 32, lattice rows that wrap inside a store, partial channel tiles, every tile shape, the compounds."""
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
    Attrs(1, 16, 1, 1, 16, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),        # no sibling inside the image
    Attrs(2, 48, 5, 8, 80, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),        # odd rows, even columns
    Attrs(1, 144, 12, 7, 32, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),
    Attrs(3, 272, 9, 33, 48, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),      # five channel tiles, 255 positions
    Attrs(1, 16, 2, 130, 528, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),     # one lattice row of 65
    Attrs(2, 256, 17, 15, 512, 1, 1, 2, 2, 1, 1, 0, 0, 0, 0),
    Attrs(1, 64, 9, 12, 64, 1, 1, 3, 1, 1, 1, 0, 0, 0, 0),       # other blocks of siblings
    Attrs(1, 64, 8, 9, 64, 1, 1, 1, 2, 1, 1, 0, 0, 0, 0),
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("tile", [None, "0", "3", "5", "6"])      # None: the default kernel, which small nodes share with test_gpu_resident.py
def test_zero_siblings(case, tile, monkeypatch):
    monkeypatch.setenv("NGC_FWD_FEW", "0")
    if tile:
        monkeypatch.setenv("NGC_G1_VARIANT", tile)
    a = CASES[case]
    x, w, b, dy = _tensors(a, "bf16", 17000 + case)
    run = Run(a, "bf16", BLK, BLK, True)
    ref = oracle.conv_bwd_data_gather(a, dy, w)
    assert oracle.max_normalised_error(run.bwd_data(dy, w), ref) <= bound("bf16", "act")
    _check_backward_compounds(run, a, x, w, dy, ref, bound("bf16", "act"))
