"""Which kernel a call runs, asked on the host: the names tell the kernels apart, the switches that force one are named for it."""
import pytest

import paper_1801_08058_amd as ng

FWD, BWD, WGRAD, DB = ng.NGC_OP_FWD, ng.NGC_OP_BWD_DATA, ng.NGC_OP_BWD_FILTERS, ng.NGC_OP_BWD_DATA_DB
NCHW, BLK = ng.NGC_NCHW, ng.NGC_NCHW16C


def node(n, c, h, w, k, r, s=None, stride=1, dtype="f32", xl=NCHW, yl=None):
    s = r if s is None else s
    pad = ((r - 1) // 2 if stride == 1 or r > 2 else 0, (s - 1) // 2 if stride == 1 or s > 2 else 0)
    return ng.make_desc(n, c, h, w, k, r, s, (stride,) * 2, (1, 1), pad, pad, ng.NGC_F32 if dtype == "f32" else ng.NGC_BF16,
                        xl, xl if yl is None else yl)


def node3(n, c, d, h, w, k, t, r, s, stride=1):
    pad = (t // 2, r // 2, s // 2)
    return ng.make_desc3(n, c, d, h, w, k, t, r, s, (stride,) * 3, (1, 1, 1), pad, pad, ng.NGC_BF16, BLK, BLK)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_names_of_the_nodes_off_the_blocked_kernels(dtype, monkeypatch):
    d, wide = node(2, 7, 13, 11, 33, 3, dtype=dtype), node(1, 3, 12, 9, 5, 4, 8, dtype=dtype)        # 9 taps, 32 taps
    for stream, name in ((0, "direct:gather"), (1, "direct:stream"), (2, "direct:stream")):
        monkeypatch.setenv("NGC_STREAM", str(stream))
        monkeypatch.setenv("NGC_WGRAD_STREAM", str(stream))
        assert [ng.ngc_conv_kernel(d, op) for op in (FWD, BWD, WGRAD)] == [name] * 3
        assert ng.ngc_conv_kernel(wide, FWD) == ng.ngc_conv_kernel(wide, BWD) == "direct:gather"
        assert ng.ngc_conv_variant(d, FWD) == "direct:gather"                                        # the variant stays
    monkeypatch.setenv("NGC_GATHER_TILE", "0")
    assert [ng.ngc_conv_kernel(d, op) for op in (FWD, BWD, WGRAD)] == ["direct"] * 3


def test_names_of_nodes_with_few_output_tiles(monkeypatch):
    d, one = node(1, 256, 14, 14, 256, 3, dtype="bf16", xl=BLK), node(1, 256, 14, 14, 256, 1, dtype="bf16", xl=BLK)
    d3, flat = node3(1, 64, 4, 7, 7, 64, 3, 3, 3), node3(1, 64, 4, 7, 7, 64, 1, 1, 1)
    for few, tail in (("0", ""), ("1", ":few"), ("2", ":few")):
        monkeypatch.setenv("NGC_FWD_FEW", few)
        for op in (FWD, BWD, DB):
            assert ng.ngc_conv_kernel(d, op) == "strip_bf16" + tail
            assert ng.ngc_conv_kernel(one, op) == "gemm1x1_bf16" + tail
        for op in (FWD, BWD):
            assert ng.ngc_conv3d_kernel(d3, op) == "strip3_bf16" + tail
            assert ng.ngc_conv3d_kernel(flat, op) == "rank2:gemm1x1_bf16" + tail
            assert ng.ngc_conv3d_variant(d3, op) == "strip3_bf16"


def test_other_kernels_keep_their_variant_names():
    for d in (node(64, 64, 56, 56, 64, 3, dtype="bf16", xl=BLK), node(8, 64, 56, 56, 64, 3, dtype="bf16"), node(64, 256, 56, 56, 64, 1, dtype="bf16", xl=BLK)):
        for op in (FWD, WGRAD):
            assert ng.ngc_conv_kernel(d, op) == ng.ngc_conv_variant(d, op)
    bad = ng.make_desc(0, 1, 1, 1, 1, 1, 1)
    assert ng.ngc_conv_kernel(bad, FWD) == "invalid"


def test_fp32_backprop_data_takes_the_kernel_that_is_expected_to_be_faster():
    """Stride 1: nodes whose two kernels differ by a tenth or more where both were timed, on either side of the choice."""
    gather = [(8, 64, 45, 37, 96, 3), (18, 62, 19, 45, 29, 5), (2, 105, 62, 52, 46, 5), (28, 41, 19, 26, 49, 5), (15, 49, 54, 39, 128, 3)]
    stream = [(2, 16, 16, 16, 32, 3), (22, 12, 16, 42, 157, 5), (12, 33, 27, 20, 160, 5), (9, 88, 24, 25, 127, 5), (8, 3, 40, 40, 32, 3)]
    for a in gather:
        assert ng.ngc_conv_kernel(node(*a), BWD) == "direct:gather", a
    for a in stream:
        assert ng.ngc_conv_kernel(node(*a), BWD) == "direct:stream", a


def tile_of(d, monkeypatch):
    """Tile of the kernel for few output tiles that backprop-data gets: the rows of channel sums of its bias gradient tell."""
    ws = {}
    for few in ("1", "2", None):
        monkeypatch.setenv("NGC_FWD_FEW", few) if few else monkeypatch.delenv("NGC_FWD_FEW")
        assert ng.ngc_conv_kernel(d, BWD).endswith(":few")
        ws[few] = ng.ngc_conv_workspace_bytes(d, DB)
    assert ws["1"] != ws["2"]
    return 32 if ws[None] == ws["1"] else 64


def test_nodes_with_few_output_tiles_take_what_is_expected_to_be_faster(monkeypatch):
    """Many taps and more than one round of 32 x 32 tiles: those take up to 1.2 times as long as the strip kernel, 64 x 64 ones, where
    there are enough of them, two thirds of its time.  One round or few taps: the small ones."""
    for a in ((4, 64, 40, 40, 48, 5), (3, 192, 27, 25, 48, 5)):
        assert tile_of(node(*a, dtype="bf16", xl=BLK), monkeypatch) == 64, a
    for a in ((1, 256, 14, 14, 256, 3), (8, 208, 7, 7, 208, 1, 7), (1, 1024, 14, 14, 256, 1), (2, 288, 21, 30, 1968, 1, 1, 2)):
        assert tile_of(node(*a, dtype="bf16", xl=BLK), monkeypatch) == 32, a
    for a in ((1, 224, 42, 31, 48, 5), (1, 272, 32, 32, 48, 5)):
        assert ng.ngc_conv_kernel(node(*a, dtype="bf16", xl=BLK), BWD) == "strip_bf16", a


SPLITS = [
    # n  c   d   h   w   k  t  r  s   bytes of partial sums, which tell the split; us so, and by a rule in the tiles' number
    ((8, 64, 16, 56, 56, 128, 3, 3, 3), 31850496),       # 190.2, 206.6
    ((6, 80, 28, 28, 22, 32, 3, 3, 3), 9289728),         # 38.8, 50.4
    ((15, 112, 6, 16, 28, 96, 3, 3, 3), 26542080),       # 42.7, 54.2
    ((2, 96, 8, 44, 33, 80, 2, 3, 3), 13934592),         # 26.3, 32.4
    ((8, 192, 20, 30, 20, 96, 2, 3, 3), 27869184),       # 85.7, 103.5
]


def test_rank3_backprop_filters_split_positions_by_expected_time():
    for a, parts_bytes in SPLITS:
        d = node3(*a)
        assert ng.ngc_conv3d_kernel(d, WGRAD) == "wgrad_gemm3_bf16:taps", a
        assert ng.ngc_conv3d_workspace_bytes(d, WGRAD) == parts_bytes, a


def test_one_tap_backprop_filters_lengthen_chunks_that_do_not_fit_an_xcd(monkeypatch):
    """384 -> 384 at 28x28: 9 tiles of 128 x 128, of which an XCD holds three chunks' worth: 24 chunks instead of 28.  512 -> 512: 31 chunks of 32."""
    for c, ordered, other in ((384, 24 * 9 << 16, 28 * 9 << 16), (512, 31 * 16 << 16, 31 * 16 << 16)):
        d = node(64, c, 28, 28, c, 1, dtype="bf16", xl=BLK)
        assert ng.ngc_conv_kernel(d, WGRAD) == "wgrad_gemm_bf16"
        assert ng.ngc_conv_workspace_bytes(d, WGRAD) == ordered
        monkeypatch.setenv("NGC_WGG_XCD", "0")
        assert ng.ngc_conv_workspace_bytes(d, WGRAD) == other
        monkeypatch.delenv("NGC_WGG_XCD")


LIMITS = [
    # n  c  h   w   k  r  stride, dtype, layout, op; us on the gather GEMM and straight to registers
    ((26, 126, 41, 22, 67, 5), 2, "f32", NCHW, BWD, 49.4, 64.7),
    ((10, 8, 29, 9, 152, 5), 2, "f32", NCHW, BWD, 25.1, 13.0),
    ((4, 90, 42, 19, 143, 5), 1, "f32", NCHW, FWD, 78.6, 31.6),
    ((31, 59, 26, 19, 65, 5), 2, "f32", NCHW, FWD, 56.8, 23.0),
    ((32, 216, 49, 8, 148, 3), 1, "bf16", NCHW, FWD, 60.1, 83.7),
    ((2, 233, 12, 52, 212, 3), 1, "bf16", NCHW, FWD, 50.2, 21.6),
    ((23, 43, 36, 33, 91, 3), 1, "bf16", NCHW, BWD, 26.9, 37.3),
    ((4, 6, 19, 35, 166, 3), 1, "bf16", NCHW, BWD, 19.2, 12.1),
    ((14, 80, 59, 17, 50, 3), 1, "bf16", BLK, FWD, 24.5, 48.1),
    ((4, 108, 10, 18, 74, 3), 2, "bf16", BLK, FWD, 22.1, 12.6),
    ((16, 166, 14, 45, 158, 3), 1, "bf16", BLK, BWD, 107.0, 197.9),
    ((3, 14, 21, 7, 232, 3), 2, "bf16", BLK, BWD, 18.1, 13.0),
    ((4, 130, 56, 35, 219, 1), 1, "bf16", NCHW, WGRAD, 11.1, 13.4),      # 128 channels or more on both sides
    ((22, 155, 24, 22, 90, 1), 1, "bf16", NCHW, WGRAD, 10.0, 9.5),
]


def test_large_nodes_off_the_blocked_kernels_keep_the_gather_gemm():
    for a, stride, dtype, layout, op, gather, stream in LIMITS:
        assert ng.ngc_conv_kernel(node(*a, stride=stride, dtype=dtype, xl=layout), op) == ("direct:gather" if gather < stream else "direct:stream"), a


@pytest.mark.parametrize("c, k, h, n, op, taken", [
    (416, 192, 27, 8, ng.NGC_OP_FWD, True), (416, 128, 27, 8, ng.NGC_OP_FWD, False), (208, 192, 27, 8, ng.NGC_OP_FWD, False),
    (256, 512, 56, 64, ng.NGC_OP_FWD, True), (256, 512, 28, 24, ng.NGC_OP_FWD, False), (528, 192, 27, 8, ng.NGC_OP_FWD, False),
    (256, 512, 56, 4, ng.NGC_OP_BWD_DATA, True), (256, 512, 56, 64, ng.NGC_OP_BWD_DATA, False), (64, 144, 56, 8, ng.NGC_OP_BWD_DATA, False),
])
def test_resident_filters_choice(c, k, h, n, op, taken):
    d = ng.make_desc(n, c, h, h, k, 1, 1, (2, 2), w_layout=ng.NGC_BLOCKED_FWD if op == ng.NGC_OP_FWD else ng.NGC_BLOCKED_BWD)
    assert ng.ngc_conv_kernel(d, op).endswith(":resident") == taken


def test_resident_filters_leave_nodes_to_the_gemm_that_it_runs_faster():
    """1x1 nodes that were timed with both kernels, a tenth or more apart: strides, channels of x and y, positions."""
    fwd = [((2, 1), 496, 144, 18496, False), ((2, 1), 400, 160, 19778, False), ((1, 2), 496, 144, 18496, True)]
    bwd = [((2, 2), 352, 48, 5236, False), ((2, 2), 480, 16, 3072, False), ((2, 2), 368, 176, 4805, False),
           ((2, 2), 64, 80, 27848, False), ((2, 2), 80, 400, 12240, True), ((2, 2), 208, 240, 7290, True), ((2, 2), 256, 48, 3600, True)]
    for op, wl, nodes in ((FWD, ng.NGC_BLOCKED_FWD, fwd), (BWD, ng.NGC_BLOCKED_BWD, bwd)):
        for stride, c, k, m, taken in nodes:
            d = ng.make_desc(1, c, stride[0], stride[1] * m, k, 1, 1, stride, w_layout=wl)
            assert ng.ngc_conv_kernel(d, op) == "gemm1x1_bf16" + (":resident" if taken else ""), (stride, c, k, m)


def test_waves_that_split_the_reduction_take_long_reductions_on_small_images():
    """Nodes that were timed with both kernels, on either side of the choice."""
    waves = [(128, 512, 7, 7, 512, 3), (32, 512, 14, 14, 512, 3), (77, 256, 15, 9, 416, 5)]
    strip = [(64, 64, 56, 56, 64, 3), (64, 128, 28, 28, 128, 3), (61, 112, 32, 16, 304, 3)]
    for a in waves + strip:
        assert ng.ngc_conv_kernel(node(*a, dtype="bf16", xl=BLK), FWD) == "strip_bf16" + (":waves" if a in waves else ""), a


def test_waves_that_split_the_reduction_leave_nodes_to_the_strip_kernel_that_it_runs_faster():
    """Nodes that took a sixth more with the waves, operands from memory, and some that took a sixth less."""
    strip = [(112, 336, 10, 16, 288, 2, 2, BWD), (32, 128, 29, 37, 272, 1, 3, BWD), (51, 800, 10, 10, 272, 3, 1, BWD), (99, 80, 17, 17, 192, 3, 3, BWD),
             (29, 224, 22, 7, 768, 3, 3, FWD), (28, 192, 13, 20, 464, 3, 3, FWD), (61, 304, 6, 23, 400, 3, 3, FWD), (69, 800, 15, 15, 320, 3, 1, FWD)]
    waves = [(84, 800, 24, 7, 192, 3, 3, FWD), (34, 944, 22, 22, 112, 3, 3, FWD), (64, 256, 14, 14, 256, 3, 3, FWD), (128, 512, 7, 7, 512, 3, 3, BWD)]
    for n, c, h, w, k, r, s, op in strip + waves:
        d = ng.make_desc(n, c, h, w, k, r, s, (1, 1), (1, 1), *[(1 if r == 2 else r // 2, 1 if s == 2 else s // 2)] * 2,
                         w_layout=ng.NGC_BLOCKED_FWD if op == FWD else ng.NGC_BLOCKED_BWD)
        assert ng.ngc_conv_kernel(d, op) == "strip_bf16" + (":waves" if (n, c, h, w, k, r, s, op) in waves else ""), (n, c, h, w, k, r, s, op)


def test_stages_of_a_waves_own_leave_short_reductions_to_common_stages():
    """Nodes that took a twentieth more with stages of a wave's own, operands from memory, and some that took a twentieth less."""
    common = [(1, 944, 26, 10, 224, 1, 9, (1, 2)), (2, 928, 7, 14, 208, 3, 3, (1, 1)), (1, 288, 32, 9, 576, 3, 3, (1, 1)), (3, 416, 14, 4, 528, 3, 3, (1, 1)),
              (7, 816, 9, 5, 304, 3, 3, (1, 1)), (4, 704, 14, 10, 272, 3, 3, (2, 2))]
    own = [(66, 64, 29, 29, 544, 3, 3, (1, 1)), (51, 256, 19, 19, 176, 3, 3, (1, 2)), (43, 432, 13, 13, 176, 3, 3, (1, 1)), (128, 512, 7, 7, 512, 3, 3, (1, 1))]
    for n, c, h, w, k, r, s, stride in common + own:
        d = ng.make_desc(n, c, h, w, k, r, s, stride, (1, 1), (r // 2, s // 2), (r // 2, s // 2))
        assert ng.ngc_conv_kernel(d, WGRAD).endswith(":taps_own") == ((n, c, h, w, k, r, s, stride) in own), (n, c, h, w, k, r, s, stride)


@pytest.mark.parametrize("n,c,h,w,k", [(112, 48, 105, 22, 64), (75, 16, 80, 19, 176), (117, 16, 79, 11, 160), (109, 16, 103, 30, 144)])
def test_parts_of_stages_of_a_waves_own_fill_every_xcd_once(n, c, h, w, k):
    """Parts in multiples of 8 or 64 and more are dealt to the 8 XCDs, whose 32 compute units hold so many (part, tile) pairs at a time."""
    d = ng.make_desc(n, c, h, w, k, 3, 3, (1, 1), (1, 1), (1, 1), (1, 1))
    tiles = (k + 63) // 64 * (c // 16)
    parts = ng.ngc_conv_workspace_bytes(d, WGRAD) // (tiles * 36864)
    assert ng.ngc_conv_kernel(d, WGRAD).endswith(":taps_own") and parts >= 64
    assert (parts + 7) // 8 * tiles <= 32


def test_backprop_filters_on_blocked_copies_need_no_more_workspace_for_stages_of_a_waves_own(monkeypatch):
    """The copies and the partials of such a node share the array of ngc_conv_bwd_filters_noalloc: what fitted it fits it still."""
    smaller = 0
    for n, c, hw, k in [(64, 256, 14, 256), (16, 144, 21, 448), (64, 128, 9, 128), (30, 96, 17, 192), (100, 64, 11, 64), (6, 256, 28, 256)]:
        ws = {}
        for own in (None, "0"):
            monkeypatch.setenv("NGC_WGRAD_OWN", own) if own else monkeypatch.delenv("NGC_WGRAD_OWN", raising=False)
            ng.ngc_reload_switches()
            ws[own] = [ng.ngc_conv_workspace_bytes(node(n, c, hw, hw, k, 3, dtype="bf16", xl=l), WGRAD) for l in (NCHW, BLK)]
        assert ws[None][0] <= ws["0"][0]
        smaller += ws[None][1] > ws["0"][1]
    assert smaller                                                       # on blocked tensors more parts are taken
