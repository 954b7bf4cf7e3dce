"""The pass that makes both gradients, at the edges of its panel sizes: the K x 64 panel of dL/dZ is staged in 2, 6 or 7
pieces per thread of 12 waves and in 6 or 10 of 16 waves, so K around 96, 288, 320 and 384, and the largest; the rows of
the transpose have 0 to K entries (whole and broken batches of 16), the second tile block is ragged.  Tolerance: the
F(4x4,3x3) contract of the other backward tests, 1e-4 of the largest value."""
import numpy as np
import pytest

from paper_1702_08597_amd import synth
from test_gpu_backward_parity import check, relerr, run_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 15, 16, 17, 96, 97, 288, 289, 320, 321, 384, 385, 638])
def test_both_gradients_at_panel_edges(K):
    N, C, H, W, m = 5, 6, 13, 13, 4
    rng = np.random.default_rng(K)
    # one dense channel, one empty one, the rest in between
    mask = rng.random((36, K, C)) < np.array([1.0, 0.0, 0.05, 0.1, 0.3, 0.6])
    rp, ci, va = synth.dense_to_csr(mask, (rng.standard_normal(mask.shape) * 0.05).astype(np.float32))
    x = synth.activations(N, C, H, W, K)
    G = rng.standard_normal((N, K, H, W)).astype(np.float32)
    check(N, C, H, W, K, m, 1, x, rp, ci, va, G)
    # without dL/dW_F the same dL/dI comes from the product alone
    both, alone = (run_backward(N, C, H, W, K, m, 1, x, rp, ci, va, G, want_dvals=w)[0] for w in (True, False))
    assert relerr(both, alone.astype(np.float64)) == 0.0
