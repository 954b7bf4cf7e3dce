"""The rows of a tile block go to LDS in dwords where a part of an image is short and in quads where it is longer than 192
floats, one to many images to a block; a span's last one to three floats travel by themselves.  Widths and heights
around that line and around whole quads and whole rounds of loads; odd planes put the channels on every alignment.
Tolerance: dL/dZ and the gradients against the oracle, the contract of the other backward tests, 1e-4 of the largest
value for F(4x4,3x3), 1e-5 for F(2x2,3x3)."""
import numpy as np
import pytest

from paper_1702_08597_amd import synth
from test_gpu_backward_parity import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(13, 13), (14, 14), (15, 13), (16, 12), (12, 17), (17, 19), (21, 21), (29, 23), (31, 33),
                                 (56, 56), (9, 113), (57, 59), (200, 5), (5, 203), (1, 257)])
@pytest.mark.parametrize("m", [2, 4])
def test_staged_rows_of_every_length(H, W, m):
    N, C, K, P = 5, 5, 6, (m + 2) ** 2
    rng = np.random.default_rng(H * 1000 + W)
    rp, ci, va = synth.bernoulli_weights(P, K, C, 0.4, H + W)
    x = synth.activations(N, C, H, W, H * W)
    G = rng.standard_normal((N, K, H, W)).astype(np.float32)
    # the forward pass inside leaves I_F, the gradient of the weights reads it, dL/dI reads the staged dL/dO
    check(N, C, H, W, K, m, 1, x, rp, ci, va, G)
