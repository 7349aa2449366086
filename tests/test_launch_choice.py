"""Which kernels the host path chooses: the rules on sizes, without a GPU."""
import os
import re

import pytest

from launch_recorder import record
from paper_2512_14080_amd import binding as B

pytestmark = pytest.mark.skipif(not os.path.exists(B.LIB_PATH), reason="libsonicmoe.so not built")


def names(launches):
    return [l[0] for l in launches]


def test_few_token_router_within_32_bit_offsets(tmp_path):
    """W_r of more than 2^32 values: not the few-token router, whose offsets have 32 bits."""
    small, large = record([{"call": "route", "dims": (1, d, 64, 1024, 8)} for d in (1 << 20, (1 << 22) + 128)], tmp_path)
    assert "StreamRouter" in names(small)[0]
    assert not any("StreamRouter" in n for n in names(large)) and "OpRouter" in names(large)[0]


@pytest.mark.parametrize("dims", [(32768, 1536, 256, 128, 8), (1000, 768, 1024, 32, 2), (13676, 2304, 320, 8, 2)])
@pytest.mark.parametrize("which", [B.MOE_WS_FWD, B.MOE_WS_BWD])
def test_workspace_size_does_not_depend_on_the_device(tmp_path, dims, which):
    """A workspace sized on one device (or without one) serves the call on any other."""
    sizes = [record([{"call": "ws", "dims": dims, "which": which, "cus": c}], tmp_path)[0] for c in (256, 32, 64, 304)]
    assert len(set(sizes)) == 1, sizes


def test_router_gradient_splits_without_dbias(tmp_path):
    """dW_r alone has 32 tiles of rows at d = 4096, in eight splits (one per CU); with the row block of dbias there
    are 33, in seven."""
    call = {"call": "bwd", "dims": (32768, 4096, 512, 128, 8)}
    for dbias, splits in ((False, 8), (True, 7)):
        launches, = record([{**call, "dbias": dbias}], tmp_path)
        dwr, = [l for l in launches if "OpDWr" in l[0]]
        assert dwr[1] == -(-splits * (33 if dbias else 32) // 8) * 8


def test_projections_of_a_rounded_routing(tmp_path):
    """Experts rounded up to m_tile rows have that many, whatever the mean of the token choice: above the streaming
    projections' range the tiled ones run."""
    dims = (512, 1536, 256, 256, 8)  # mean 16
    forms = [None, (16, "nearest"), (16, "up"), (32, "nearest"), (128, "up"), (256, "up")]
    calls = [{"call": "fwd", "dims": dims, **({"round": f} if f else {})} for f in forms]
    stream = [["StreamUp" in "".join(names(l)), "StreamDown" in "".join(names(l))] for l in record(calls, tmp_path)]
    assert stream == 3 * [[True, True]] + 3 * [[False, False]]


@pytest.mark.parametrize("T,E,K,rows", [(1000, 512, 8, 32), (4000, 2048, 4, 32), (4000, 256, 1, 0), (2000, 256, 1, 32),
                                        (17, 8, 8, 32), (16, 16, 16, 16), (200, 512, 4, 16)])
def test_streaming_grid_holds_a_hot_experts_groups(tmp_path, T, E, K, rows):
    """The experts' first groups of `rows` rows and all that a skewed router can add (K hot experts with every token),
    each with a workgroup of its own; not from 12 rows per expert on where an expert can have many groups (rows 0)."""
    launches, = record([{"call": "fwd", "dims": (T, 1536, 256, E, K)}], tmp_path)
    if not rows:
        assert not any("stream_gemm_kernel" in l[0] for l in launches)
        return
    for l in launches[:2]:
        assert "stream_gemm_kernel" in l[0] and l[3] == 1
        assert E + K * ((T - 1) // rows) <= l[2] <= E + T * K // rows


@pytest.mark.parametrize("dims,scores_in,few", [
    ((1024, 128, 64, 64, 8), False, True), ((2048, 128, 64, 64, 8), False, False), ((2048, 768, 64, 64, 8), False, True),
    ((4096, 768, 64, 64, 8), False, False), ((4096, 128, 64, 64, 2), False, True), ((4096, 128, 64, 128, 8), False, False),
    ((4096, 128, 64, 256, 8), False, True), ((4096, 128, 64, 64, 16), False, True), ((256, 128, 64, 8, 8), True, True),
    ((512, 128, 64, 8, 8), True, False), ((16, 128, 64, 8, 8), True, True), ((17, 128, 64, 8, 8), True, True),
])
def test_few_token_routing_for_counts_only(tmp_path, dims, scores_in, few):
    """Where only the counts are wanted, the few-token form is left where its metadata costs more than the bitmap's;
    the complete routing of the same sizes keeps it."""
    flags = B.MOE_ROUTE_SCORES_IN if scores_in else 0
    full, counts = record([{"call": "route", "dims": dims, "flags": flags | f} for f in (0, B.MOE_ROUTE_COUNTS_ONLY)],
                          tmp_path)
    assert any("topk_few" in n for n in names(full))
    assert any("topk_few" in n for n in names(counts)) == few
    assert any("expert_scan" in n for n in names(counts)) == (not few)


@pytest.mark.parametrize("d,n,plain", [(1536, 256, {"OpUp", "OpDown", "OpDH", "OpDXt"}), (1664, 448, set()),
                                       (2048, 512, {"OpUp", "OpDH"}), (1024, 1024, {"OpDown", "OpDH", "OpDXt"})])
def test_whole_tiles_in_row_order(tmp_path, d, n, plain):
    """256-wide tiles that all lie within the matrix, fewer than eight to a row, take the kernels without column limits
    and blocked order; an uneven last tile or longer rows the general ones."""
    fwd, bwd = record([{"call": c, "dims": (32768, d, n, 128, 8), "dbias": True} for c in ("fwd", "bwd")], tmp_path)
    found = {}
    for name in names(fwd + bwd):
        m = re.search(r"(OpUp|OpDown|OpDH|OpDXt)INS_7GemmCfgILi256ELi256E.*?EEE(Li0E)?Lb([01])E", name)
        if m:
            found[m.group(1)] = m.group(3) == "1"
    assert set(found) == {"OpUp", "OpDown", "OpDH", "OpDXt"}
    assert {k for k, v in found.items() if v} == plain


@pytest.mark.parametrize("dims,form,width", [
    ((643, 1792, 448, 88, 3), None, 256), ((643, 1792, 448, 88, 3), (256, "nearest"), 64),  # about eight experts left
    ((3084, 4096, 512, 128, 8), None, 64), ((3084, 4096, 512, 128, 8), (128, "up"), 256),  # one m-tile each
    ((512, 1536, 256, 128, 4), (256, "up"), 128), ((512, 1536, 256, 128, 4), (256, "down"), 64),
    ((32768, 1536, 256, 128, 8), None, 256), ((32768, 1536, 256, 128, 8), (128, "nearest"), 256),
])
def test_tile_width_follows_the_rounding(tmp_path, dims, form, width):
    """dH's tiles by the m-tiles that the rounding leaves, not by those of the token choice."""
    call = {"call": "bwd", "dims": dims, "dbias": True, **({"round": form} if form else {})}
    launches, = record([call], tmp_path)
    dh, = [n for n in names(launches) if "OpDH" in n]
    assert f"GemmCfgILi256ELi{width}E" in dh


def test_kernels_of_the_fused_router_tests(tmp_path):
    """The shapes that test_gpu_router_topk names fused run the fused router (and with MOE_ROUTE_SEPARATE_TOPK the
    router GEMM and the lane-per-token kernel); its few-token ones the few-token kernels, with either flag."""
    from test_gpu_router_topk import FEW, FUSED
    shapes = [(c.T, c.d, c.n, c.E, c.K) for c in FUSED + FEW]
    got = record([{"call": "route", "dims": s, "flags": f} for s in shapes for f in (0, B.MOE_ROUTE_SEPARATE_TOPK)],
                 tmp_path)
    for i, s in enumerate(shapes):
        one, two = names(got[2 * i]), names(got[2 * i + 1])
        if i < len(FUSED):
            assert "OpRouterTopk" in one[0] and "OpRouterI" in two[0] and "topk_lane" in two[1], s
        else:
            assert one == two and "StreamRouter" in one[0] and "topk_few" in one[1], s


def test_kernels_of_the_wide_selections(tmp_path):
    """E > 256 with more than 4096 tokens, and E > 1024 with any number: the wave-per-token kernel over 64-token words."""
    shapes = [(4200, 264, 3), (4200, 1024, 8), (700, 2056, 16), (700, 4096, 16), (4200, 16, 10), (4200, 24, 3)]
    for s, l in zip(shapes, record([{"call": "route", "dims": (T, 128, 64, E, K), "flags": B.MOE_ROUTE_SCORES_IN}
                                    for T, E, K in shapes], tmp_path)):
        assert ("topk_route" if s[1] > 256 else "topk_lane") in names(l)[0], s
