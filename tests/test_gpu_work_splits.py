"""Parity of the layer with the oracle at the sizes where the kernels' work
splits change: the edges of tiles and chunks, remainders, the smallest and the
largest sizes of a variant's range.  Tolerances as in test_gpu_parity."""
import numpy as np
import pytest

from paper_2512_14080_amd import workloads as W
from test_gpu_parity import check_layer, expert_biases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,shift", [(300, -40.0), (520, 0.0), (1400, 1.5)])
def test_expert_bias_gradients_over_row_tiles(T, shift):
    """db1 and db2 are summed per 256-row tile and then over an expert's tiles:
    experts without rows, with one partial tile, with full tiles only (one
    expert takes every token; T = 512 of them make two full tiles) and with
    both.  Column counts off the 512-column chunks."""
    cfg = W.MoEConfig("colsum", T=T, d=640, n=192, E=8, K=2, m_tile=64)
    bias = np.array([0, 0.3, shift, 0.6, 40.0, 0, -0.5, 1.0], np.float32)
    T = 512 if T == 520 else T
    layer, R = check_layer(cfg, seed=31, T=T, bias=bias, eb=expert_biases(cfg, 31))
    assert R.counts[4] == T and (shift > -40 or R.counts[2] == 0)


def test_weight_gradients_of_equal_experts():
    """Experts of equal length a little over the 2048-row chunk: dW1 (256
    tiles, whole rounds of the CUs) leaves them whole, dW2 (128 tiles) cuts
    each into 2048 rows and a 64-row remainder."""
    cfg = W.MoEConfig("equal", T=2112, d=4096, n=256, E=8, K=8, m_tile=128)
    layer, R = check_layer(cfg, seed=32)
    assert (R.counts == 2112).all()


@pytest.mark.parametrize("T,d,n,E,K,zipf", [
    (1, 128, 64, 8, 1, 0.0),      # one row; fewer k steps (n: 2, d: 4) than waves
    (3, 384, 192, 40, 3, 0.0),    # one row block, the last of the k splits uneven
    (10, 896, 320, 8, 8, 0.0),    # one row block of 10 rows, K = E
    (16, 768, 256, 8, 8, 0.0),    # its largest T
    (17, 768, 256, 8, 8, 0.0),    # two row blocks
    (11, 768, 256, 8, 8, 0.0),
    (20, 256, 128, 16, 16, 0.0),  # two row blocks at their largest mean (20)
    (21, 256, 128, 16, 16, 0.0),  # four row blocks
    (128, 640, 192, 8, 4, 0.0),   # four at their largest mean (64), rows past one group
    (129, 640, 192, 8, 4, 0.0),   # the tiled GEMMs
    (150, 256, 64, 120, 8, 1.5),  # skewed: empty experts, and experts with many groups of 16 rows
    (300, 128, 64, 2056, 4, 1.5),  # the same over more experts than one pass of the group search holds
    (600, 640, 192, 320, 8, 1.5),  # of 32 rows
    (600, 384, 192, 320, 1, 1.5),  # of 16 rows (mean 2)
    (140, 640, 192, 24, 8, 3.0),  # of 64 rows
])
@pytest.mark.parametrize("biased", [False, True])
def test_few_rows_per_expert(T, d, n, E, K, zipf, biased):
    """The streaming projections (few rows per expert) on both sides of their
    row-block rules, with and without expert biases."""
    cfg = W.MoEConfig("few", T=T, d=d, n=n, E=E, K=K, m_tile=16, zipf_s=zipf)
    layer, R = check_layer(cfg, seed=33, eb=expert_biases(cfg, 33) if biased else None)
    if zipf:
        assert R.counts.max() > 128 and R.counts.min() == 0


@pytest.mark.parametrize("T,d,E,K,mode", [
    (1, 128, 8, 1, None),        # one token: one workgroup for top-K and metadata; four k steps
    (16, 256, 72, 3, None),      # the last T of the one-workgroup form
    (17, 256, 72, 3, None),      # the first past it
    (16, 256, 72, 3, "up"),      # the one-workgroup form for counts and transposed scores, rows left by the rounding
    (64, 1536, 128, 8, None),    # one whole word; several k slices
    (65, 384, 40, 3, None),      # a lone token in the second word
    (300, 4096, 200, 16, None),  # K > 8, E off the 64-lane groups
    (1000, 256, 264, 12, "nearest"),
    (63, 256, 24, 5, "nearest"),  # rounding on one word, its last token missing
    (4096, 128, 64, 8, None),    # the last T of the few-token form
    (4097, 128, 64, 8, None),    # the first T past it
    (200, 128, 1024, 2, "up"),   # the largest E of the form, transposed scores beyond 64 KB of LDS
    (200, 128, 1032, 2, None),   # the first E past it
    (700, 128, 2056, 4, None),   # three workgroups of rows, the last partial, each over three passes of experts
])
def test_few_token_routing(T, d, E, K, mode):
    """The routing of few tokens: its own router against the oracle's logits,
    with every integer result a function of the scores it writes (the same
    call with those scores given, and the oracle's routing of them)."""
    import oracle
    from test_gpu_parity import _torch, check_routing, oracle_routing
    from dense_reference import rel_err
    torch = _torch()
    from paper_2512_14080_amd import binding as B
    from paper_2512_14080_amd.layer import DeviceLayer
    cfg = W.MoEConfig("route", T=T, d=d, n=64, E=E, K=K, m_tile=8 if T == 16 else 16, zipf_s=0.5)
    inp = W.make_inputs(cfg, 34)
    layers = []
    for scores in (None, "given"):
        if scores:
            scores = layers[0].tc.arrays()["scores"].cpu().numpy()
        layer = DeviceLayer(inp, round_mode=mode, scores_in=scores)
        layer.route()
        torch.cuda.synchronize()
        layers.append(layer)
    L = oracle.router_logits(inp.f32("X"), inp.f32("Wr"), inp.bias, np.float32)
    a = {k: v.cpu().numpy() for k, v in layers[0].tc.arrays().items() if v is not None}
    assert rel_err(a["logits"], L) <= 1e-4
    assert rel_err(a["scores"], oracle.softmax_scores(L).astype(np.float32)) <= 1e-4
    idx, rdir, R = oracle_routing(a["scores"], K, mode, cfg.m_tile)
    for layer in layers:
        check_routing(layer, R, idx, rdir)
        t = layer.tc.arrays()
        if mode:
            np.testing.assert_array_equal(t["scores_t"].cpu().numpy(), a["scores"].T)
            member = np.zeros((T, E), bool)
            np.put_along_axis(member, idx, True, axis=1)
            np.testing.assert_array_equal(t["counts"].cpu().numpy(), member.sum(0))


def test_router_weights_past_32_bit_offsets():
    """W_r of 2^32 values and more (the few-token router's offsets have 32 bits):
    the logits come from the last row of W_r, the only one that is not zero."""
    from test_gpu_parity import _torch
    torch = _torch()
    from paper_2512_14080_amd import binding as B
    d, E = (1 << 22) + 128, 1024
    X = torch.zeros((1, d), dtype=torch.bfloat16, device="cuda")
    Wr = torch.zeros((d, E), dtype=torch.bfloat16, device="cuda")
    X[0, -1] = 1.0
    Wr[-1] = torch.arange(E, device="cuda") / 256.0  # at most 8 significant bits up to 1, rounded beyond
    D = B.dims(1, d, 64, E, 8)
    r = B.Routing(D, 8, B.MOE_ROUTING_LOGITS)
    B.moe_route(D, X, Wr, None, B.MOE_ROUTE_WRITE_LOGITS, r)
    torch.cuda.synchronize()
    assert torch.equal(r.arrays()["logits"][0], Wr[-1].float())


@pytest.mark.parametrize("T,E,K", [
    (16, 8, 8), (17, 72, 5), (70, 136, 8), (33, 264, 16), (90, 520, 7), (20, 1024, 1),
    (16, 64, 5), (40, 64, 6), (40, 136, 7), (33, 264, 8), (16, 1024, 9),  # both selects, on both sides of their rule
    (4100, 264, 8), (4100, 520, 9), (4100, 1024, 2),                      # past the few-token form
    (4100, 24, 3), (4100, 72, 7), (4100, 40, 12), (4100, 128, 8), (4100, 64, 16),  # lane per token, one wave and four
])
def test_selection_with_ties(T, E, K):
    """Given scores with many equal values, zeros of both signs and rows of one
    value: the selection still takes the lowest experts, in the oracle's order."""
    from test_gpu_parity import _torch, check_routing, oracle_routing
    torch = _torch()
    from paper_2512_14080_amd.layer import DeviceLayer
    cfg = W.MoEConfig("ties", T=T, d=128, n=64, E=E, K=K, m_tile=16)
    rng = np.random.default_rng(E + K)
    S = (rng.integers(1, 5, (T, E)) / np.float32(8)).astype(np.float32)
    S[0] = 0.25
    S[1, ::2], S[1, 1::2] = 0.0, -0.0
    S[1, E // 2] = 0.5
    layer = DeviceLayer(W.make_inputs(cfg, 35), scores_in=S)
    layer.route()
    torch.cuda.synchronize()
    idx, _, R = oracle_routing(S, K)
    np.testing.assert_array_equal(layer.tc.arrays()["topk_idx"].cpu().numpy(), idx)
    np.testing.assert_array_equal(layer.tc.arrays()["row_token"].cpu().numpy(), R.row_token)
    np.testing.assert_array_equal(layer.tc.arrays()["row_expert"].cpu().numpy(), R.row_expert)


def test_wide_tiles_on_short_loops():
    """Enough experts for the 256 x 256 tiles of every GEMM, with the loops at
    their shortest: down (k = n = 64) and dX~ (k = 2n = 128) on the split LDS
    ring, and weight gradients over experts of 0 to 4 k steps of 64 rows."""
    cfg = W.MoEConfig("ring", T=1600, d=768, n=64, E=72, K=2, m_tile=64)
    check_layer(cfg, seed=36)
    check_layer(cfg, seed=36, eb=expert_biases(cfg, 36))
    cfg = W.MoEConfig("kshort", T=1200, d=512, n=256, E=72, K=2, m_tile=64)
    bias = np.concatenate([[-40.0], np.linspace(-5.0, 1.5, cfg.E - 1)]).astype(np.float32)
    for mode in (None, "nearest"):
        layer, R = check_layer(cfg, seed=37, bias=bias, round_mode=mode)
        steps = set(int(-(-c // 64)) for c in R.counts)
        assert steps >= {0, 1, 2, 3}, steps


@pytest.mark.parametrize("T,d,n,E,K", [
    (1280, 512, 512, 16, 2),   # 16 to 24 m-tiles: narrow tiles and small dW tiles throughout
    (600, 1536, 512, 64, 4),   # 64 m-tiles x 6: between one round and one and a half of down and dX~
    (1000, 256, 1024, 32, 2),  # up 256 wide tiles, dH 128: on both sides of half a round
])
def test_narrow_tiles(T, d, n, E, K):
    check_layer(W.MoEConfig("narrow", T=T, d=d, n=n, E=E, K=K, m_tile=128), seed=38)


@pytest.mark.parametrize("T,d,n,E,K,mode", [
    (3000, 896, 192, 40, 3, None),         # dH one 256-wide tile, dW 256 x 256: columns and rows past both
    (3000, 1152, 320, 24, 4, "nearest"),   # down and dX~ 256-wide over d = 4.5 tiles, up over n = 2.5
    (9000, 1152, 448, 8, 4, None),         # the same with split experts' fp32 slabs
    (2500, 640, 64, 48, 4, None),          # n of one narrow tile
    (700, 640, 576, 8, 2, None),           # few tiles: narrow shapes with masked halves
])
@pytest.mark.parametrize("biased", [False, True])
def test_columns_off_the_wide_tiles(T, d, n, E, K, mode, biased):
    """d an odd multiple of 128 and n an odd multiple of 64: the last 256-wide
    tile of a row is partly past the matrix, in every GEMM of the layer."""
    cfg = W.MoEConfig("offgrid", T=T, d=d, n=n, E=E, K=K, m_tile=128, zipf_s=1.2 if T == 9000 else 0.0)
    check_layer(cfg, seed=39, round_mode=mode, eb=expert_biases(cfg, 39) if biased else None)
