"""Filter re-layout through LDS tiles (2-byte elements, C a multiple of 16), bit for bit: rows that end inside a tile on
either channel axis, the largest window the tiles hold; the one past it and small filters take a thread per element."""
import numpy as np
import pytest
import torch

import paper_1801_08058_amd as ng
from gpu_util import dev, filter_blocked_host, host, stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kcrs", [(1040, 1072, 1, 1), (296, 304, 3, 3), (72, 80, 5, 5), (17, 1200, 1, 7), (70, 16, 10, 12), (74, 16, 11, 11), (33, 16, 1, 1)])
@pytest.mark.parametrize("layout", [ng.NGC_BLOCKED_FWD, ng.NGC_BLOCKED_BWD])
def test_filter_tiles_bit_exact(kcrs, layout):
    K, C, R, S = kcrs
    bits = np.random.default_rng(K * 31 + C).integers(1, 0xFFFF, size=kcrs, dtype=np.uint16)
    d = ng.make_desc(1, C, 24, 24, K, R, S, pad_below=(R // 2, S // 2), pad_above=(R // 2, S // 2))
    exp = filter_blocked_host(bits, layout).reshape(-1)
    dst = torch.full((exp.size,), -1, dtype=torch.int16, device="cuda")
    ng.ngc_filter_convert(d, dev(bits), dst, layout, stream())
    torch.cuda.synchronize()
    assert np.array_equal(host(dst, np.uint16), exp)
