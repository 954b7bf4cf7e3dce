"""The weight gradient's sums in the launch of the input gradient (images of one pass of 64 tiles): both gradients asked for
together against each by itself - two launches, the same bits - and against the oracle.  Without padding a few small
images make one tile each, so a workgroup holds the planes of 64 of them: up to 66 KB of LDS."""
import numpy as np
import pytest
import torch

import oracle
from paper_1702_08597_amd import binding as sw
from paper_1702_08597_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C,H,K,m,r,pad", [
    (70, 9, 8, 10, 4, 5, 0),    # 64 planes of 8 x 8 a wave
    (67, 17, 6, 13, 4, 3, 0),   # 64 of 6 x 6
    (130, 6, 4, 9, 2, 3, 0),    # 64 of 4 x 4
    (9, 21, 7, 30, 4, 3, 1),    # sixteen images of four tiles
    (3, 20, 27, 12, 4, 5, 2),   # one image, 49 tiles
])
def test_together_and_apart(N, C, H, K, m, r, pad):
    rng = np.random.default_rng(N + C)
    P, Ho = (m + r - 1) ** 2, H + 2 * pad - r + 1
    rp, ci, va = synth.bernoulli_weights(P, K, C, 0.3, N)
    x = synth.activations(N, C, H, H, 5)
    G = rng.standard_normal((N, K, Ho, Ho)).astype(np.float32)
    xd, gd = torch.from_numpy(x).cuda(), torch.from_numpy(G).cuda()
    plan = sw.swconv_plan_create(N, C, H, H, K, m, r, pad)
    try:
        sw.swconv_set_weights(plan, rp, ci, va)
        got = {}
        for want in ("both", "din", "dvals"):
            din, dvals = torch.full_like(xd, float("nan")), torch.full((len(va),), float("nan"), device="cuda")
            sw.swconv_backward(plan, 0, xd.data_ptr(), gd.data_ptr(), 0 if want == "dvals" else din.data_ptr(),
                               0 if want == "din" else dvals.data_ptr())
            torch.cuda.synchronize()
            got[want] = din.cpu().numpy(), dvals.cpu().numpy()
    finally:
        sw.swconv_plan_destroy(plan)
    np.testing.assert_array_equal(got["both"][0].view(np.uint32), got["din"][0].view(np.uint32))
    np.testing.assert_array_equal(got["both"][1].view(np.uint32), got["dvals"][1].view(np.uint32))
    din64, dvals64, _, _ = oracle.backward_f64(x, rp, ci, va, G, K, m, r, pad, want_ZV=False)
    rtol = 1e-5 if (m, r) == (2, 3) else 1e-4
    assert np.abs(got["both"][0] - din64).max() <= rtol * np.abs(din64).max()
    assert np.abs(got["both"][1] - dvals64).max() <= rtol * np.abs(dvals64).max()
