"""Infinities at places the sums must not reach: elements of the padding, of channels and of positions past the end."""
import numpy as np
import pytest

import oracle
import paper_1801_08058_amd as ng
from oracle import Attrs
from gpu_util import Run, bound, host
from test_gpu_parity import _tensors

pytestmark = pytest.mark.gpu
NCHW, BLK = ng.NGC_NCHW, ng.NGC_NCHW16C


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tile", [1, 2, 3])
def test_infinite_filter_leaves_the_padding_lanes_zero(dtype, tile, monkeypatch):
    """Reduction indices past the end meet output channels past the end: both read zero, not filter element 0."""
    monkeypatch.setenv("NGC_GATHER_TILE", str(tile))
    a = Attrs(1, 5, 6, 6, 20, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1)
    x, w, b, dy = _tensors(a, dtype, 15000)
    w[0, 0, 0, 0] = np.inf
    run = Run(a, dtype, BLK, BLK, False)
    bits = np.uint16 if dtype == "bf16" else np.uint32
    y = run.fwd(x, w, bias=b, relu=False)
    assert np.all(host(run.last_raw, bits).reshape(1, 2, 6, 6, 16)[:, 1, :, :, 4:] == 0)
    w0 = w.copy()
    w0[0] = 0
    assert oracle.max_normalised_error(y[:, 1:], oracle.conv_fwd(a, x, w0, bias=b)[:, 1:]) <= bound(dtype, "act")
    run.bwd_data(dy, w)
    assert np.all(host(run.last_raw, bits).reshape(1, 1, 6, 6, 16)[..., 5:] == 0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tile", [1, 2, 3])
def test_infinite_input_leaves_the_padding_lanes_zero(dtype, tile, monkeypatch):
    monkeypatch.setenv("NGC_GATHER_TILE", str(tile))
    a = Attrs(1, 5, 6, 6, 20, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1)
    x, w, b, dy = _tensors(a, dtype, 15001)
    x[0, 2, 3, 3] = np.inf
    dy[0, 7, 2, 2] = -np.inf
    run = Run(a, dtype, BLK, BLK, False)
    bits = np.uint16 if dtype == "bf16" else np.uint32
    run.fwd(x, w, bias=b, relu=False)
    assert np.all(host(run.last_raw, bits).reshape(1, 2, 6, 6, 16)[:, 1, :, :, 4:] == 0)
    run.bwd_data(dy, w)
    assert np.all(host(run.last_raw, bits).reshape(1, 1, 6, 6, 16)[..., 5:] == 0)
