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
    (10, 896, 320, 8, 8, 0.0),    # one row block at its largest mean (10 rows an expert), K = E
    (11, 768, 256, 8, 8, 0.0),    # two row blocks
    (20, 256, 128, 16, 16, 0.0),  # two row blocks at their largest mean (20)
    (21, 256, 128, 16, 16, 0.0),  # four row blocks
    (128, 640, 192, 8, 4, 0.0),   # four at their largest mean (64), rows past one group
    (129, 640, 192, 8, 4, 0.0),   # the tiled GEMMs
    (150, 256, 64, 120, 8, 1.5),  # skewed: empty experts, and experts with many groups of 16 rows
])
@pytest.mark.parametrize("biased", [False, True])
def test_few_rows_per_expert(T, d, n, E, K, zipf, biased):
    """The streaming projections (few rows per expert) on both sides of their
    row-block rules, with and without expert biases."""
    cfg = W.MoEConfig("few", T=T, d=d, n=n, E=E, K=K, m_tile=16, zipf_s=zipf)
    layer, R = check_layer(cfg, seed=33, eb=expert_biases(cfg, 33) if biased else None)
    if zipf:
        assert R.counts.max() > 128 and R.counts.min() == 0
