"""Gather GEMM kernels (fp32 tensors, channel counts off the block, first layers) against the oracle: every tile of
forward / backprop-data and of backprop-filters, one part and several, at sizes around the edges of their tiles and
steps; the split reduction without a workspace."""
import pytest
import torch

import oracle
import paper_1801_08058_amd as ng
from oracle import Attrs
from gpu_util import Run, bound, data_to_device, desc_of, stream
from test_gpu_parity import _check_all, _tensors

pytestmark = pytest.mark.gpu
NCHW, BLK = ng.NGC_NCHW, ng.NGC_NCHW16C

CASES = [
    # n  c   h   w   k   r  s  sh sw dh dw pbh pbw pah paw
    (Attrs(1, 1, 5, 5, 1, 1, 1, 1, 1, 1, 1, 0, 0, 0, 0), "f32", NCHW, NCHW),         # one output channel, one index
    (Attrs(3, 7, 13, 11, 33, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "f32", NCHW, NCHW),      # one channel past a tile
    (Attrs(2, 16, 8, 16, 64, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "f32", NCHW, NCHW),      # whole tiles, aligned filter rows
    (Attrs(2, 65, 9, 15, 31, 3, 2, 2, 3, 1, 2, 2, 0, 1, 3), "f32", NCHW, BLK),       # strides and dilation: classes without taps
    (Attrs(1, 5, 40, 37, 66, 5, 5, 4, 3, 1, 1, 2, 2, 2, 2), "f32", BLK, NCHW),       # largest stride the classes hold
    (Attrs(2, 3, 33, 35, 40, 7, 7, 2, 2, 1, 1, 3, 3, 3, 3), "bf16", NCHW, BLK),      # first layer, width off the 16-byte grid
    (Attrs(4, 40, 14, 14, 72, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1), "bf16", NCHW, NCHW),
    (Attrs(1, 3, 40, 9, 5, 31, 1, 1, 1, 1, 1, 15, 0, 15, 0), "f32", NCHW, NCHW),     # longest window
    (Attrs(1, 3, 40, 9, 5, 32, 1, 1, 1, 1, 1, 15, 0, 15, 0), "f32", NCHW, NCHW),     # one tap more: the one-thread-per-output kernels
    (Attrs(1, 2, 12, 12, 3, 3, 3, 5, 1, 1, 1, 1, 1, 1, 1), "bf16", NCHW, NCHW),      # one stride more
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("tile,wgrad", [(None, None), (1, 1001), (2, 2001), (3, 3001), (1, 1003), (2, 2002), (3, 3005)])
def test_gather_tiles(case, tile, wgrad, monkeypatch):
    a, dtype, xl, yl = CASES[case]
    if tile:
        monkeypatch.setenv("NGC_GATHER_TILE", str(tile))
        monkeypatch.setenv("NGC_GATHER_WGRAD", str(wgrad))
    names = ["direct:gather"] * 3
    if a.r > 31:
        names = ["direct"] * 3
    elif max(a.sh, a.sw) > 4:
        names[1] = "direct"
    _check_all(a, dtype, xl, yl, False, 12000 + case, names)
    assert ng.ngc_conv_variant(desc_of(a, dtype, xl, yl), ng.NGC_OP_FWD) == names[0]


@pytest.mark.parametrize("dtype,node", [
    ("f32", (2, 21, 33, 10, 128, 3, 1)),      # 660 positions in 20 parts
    ("f32", (8, 64, 45, 37, 96, 3, 1)),       # 13320 positions, partials near their limit
    ("f32", (8, 128, 14, 14, 160, 3, 1)),
    ("f32", (2, 300, 40, 40, 300, 3, 1)),     # few parts of a large dw
    ("f32", (1, 520, 36, 36, 1000, 3, 1)),    # one part: dw past the limit of the partials
    ("f32", (4, 900, 24, 24, 32, 5, 1)),      # small tiles, few parts
    ("f32", (1, 34, 14, 9, 56, 5, 1)),        # one part, eight slices
    ("f32", (16, 20, 30, 30, 12, 3, 1)),      # small tiles
    ("bf16", (15, 170, 22, 14, 147, 3, 1)),
    ("bf16", (8, 40, 28, 28, 72, 3, 1)),
])
@pytest.mark.parametrize("with_ws", [True, False])
def test_backprop_filters_sums_are_as_exact_as_the_thread_per_position_kernels(dtype, node, with_ws, monkeypatch):
    """2-norm errors against 64 bits: at most 1.35 times that of 256 chains per element and a tree (the order of the sums
    differs; one chain per element is at 1.5 to 15 times).  Each level of additions adds the square of about 2.6e-8, and
    neither order has more than a fifth more levels than the other here."""
    n, c, h, w, k, r, st = node
    d = ng.make_desc(n, c, h, w, k, r, r, (st, st), (1, 1), (r // 2, r // 2), (r // 2, r // 2), ng.NGC_F32 if dtype == "f32" else ng.NGC_BF16, NCHW, NCHW)
    monkeypatch.setenv("NGC_STAGED", "0")
    tt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(12200 + n)
    x, dy = torch.randn(n, c, h, w, generator=g, device="cuda").to(tt), (0.1 * torch.randn(n, k, h, w, generator=g, device="cuda")).to(tt)
    xp = torch.nn.functional.pad(x.double(), (r // 2,) * 4)
    dyt = dy.double().permute(1, 0, 2, 3).reshape(k, -1)
    ref = torch.stack([dyt @ xp[:, :, i : i + h, j : j + w].permute(1, 0, 2, 3).reshape(c, -1).t() for i in range(r) for j in range(r)], 2).flatten()

    def error(name):
        assert ng.ngc_conv_variant(d, ng.NGC_OP_BWD_FILTERS) == name
        dw = torch.full((k * c * r * r,), float("nan"), dtype=torch.float32, device="cuda")
        need = ng.ngc_conv_workspace_bytes(d, ng.NGC_OP_BWD_FILTERS)
        ng.ngc_conv_bwd_filters(d, x, dy, dw, torch.empty(need, dtype=torch.uint8, device="cuda") if with_ws and need else None, stream())
        torch.cuda.synchronize()
        return float((dw.double() - ref).norm() / ref.norm())

    got = error("direct:gather")
    monkeypatch.setenv("NGC_GATHER_TILE", "0")
    base = error("direct")
    print(f"case {dtype} {node} ws={with_ws}: {got:.2e} against {base:.2e}", flush=True)
    assert got <= 1.35 * base


@pytest.mark.parametrize("node,name", [((32, 3, 20, 20, 11, 3), "direct"), ((4, 100, 20, 20, 90, 3), "gather")])
def test_split_nodes_without_a_workspace_take_the_faster_kernel(node, name, monkeypatch):
    """Bit for bit the thread-per-position kernel where one part of the GEMM would leave the chip empty."""
    n, c, h, w, k, r = node
    a = Attrs(n, c, h, w, k, r, r, 1, 1, 1, 1, 1, 1, 1, 1)
    x, _, _, dy = _tensors(a, "f32", 12300 + c)
    d = desc_of(a, "f32", NCHW, NCHW)
    assert ng.ngc_conv_workspace_bytes(d, ng.NGC_OP_BWD_FILTERS) > 0
    xd, dyd, got = data_to_device(x, "f32", NCHW), data_to_device(dy, "f32", NCHW), []
    for tile in (None, "0"):
        if tile:
            monkeypatch.setenv("NGC_GATHER_TILE", tile)
        dw = torch.full((k * c * r * r,), float("nan"), dtype=torch.float32, device="cuda")
        ng.ngc_conv_bwd_filters(d, xd, dyd, dw, None, stream())
        torch.cuda.synchronize()
        got.append(dw)
    assert torch.equal(*got) == (name == "direct")
    ref = oracle.conv_bwd_filters(a, x, dy)
    assert oracle.max_normalised_error(got[0].cpu().numpy().astype("float64").reshape(k, c, r, r), ref) <= bound("f32", "dw")


def test_backprop_filters_without_a_workspace():
    """The partial sums' workspace is optional for these nodes: without it one part runs, same result to fp32 rounding."""
    a = Attrs(6, 20, 24, 24, 24, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1)
    x, w, b, dy = _tensors(a, "f32", 12100)
    d = desc_of(a, "f32", NCHW, NCHW)
    assert ng.ngc_conv_workspace_bytes(d, ng.NGC_OP_BWD_FILTERS) > 0
    dw = torch.full((a.k * a.c * 9,), float("nan"), dtype=torch.float32, device="cuda")
    ng.ngc_conv_bwd_filters(d, data_to_device(x, "f32", NCHW), data_to_device(dy, "f32", NCHW), dw, None, stream())
    torch.cuda.synchronize()
    got = dw.cpu().numpy().astype("float64").reshape(a.k, a.c, 3, 3)
    assert oracle.max_normalised_error(got, oracle.conv_bwd_filters(a, x, dy)) <= bound("f32", "dw")
    assert oracle.max_normalised_error(Run(a, "f32", NCHW, NCHW, False).bwd_filters(x, dy), got) <= bound("f32", "dw")
