"""dL/dI where tiles meet: columns are summed between lanes (and between passes of 64 tiles), rows through LDS.  Images of
one tile, one row or column of tiles, 64 and 65 tiles, several images to a pass, passes that end inside a row of tiles,
edges 1 to m pixels wide, planes of whole and broken quads, every padding, a group that is not full.  Integer data:
dL/dI equal to the oracle bit for bit for the 3x3 filters; for F(4x4,5x5), whose matrices hold fractions, 1e-4 of the
largest value as in its other tests."""
import numpy as np
import pytest
import torch

import oracle
from paper_1702_08597_amd import binding as sw
from paper_1702_08597_amd import synth

pytestmark = pytest.mark.gpu


SIZES = [(3, 3), (4, 4), (5, 5), (4, 40), (40, 4), (6, 7), (13, 13), (16, 9), (32, 32), (33, 31), (17, 52), (20, 53),
         (54, 35), (56, 56)]
KINDS = [(2, 3, 0), (2, 3, 1), (4, 3, 0), (4, 3, 1), (4, 3, 2), (4, 5, 0), (4, 5, 2)]
CASES = [(h, w, m, r, pad) for h, w in SIZES for m, r, pad in KINDS if min(h, w) + 2 * pad >= r]


@pytest.mark.parametrize("H,W,m,r,pad", CASES)
def test_patches_meet(H, W, m, r, pad):
    N, C, K, P = 7, 5, 6, (m + r - 1) ** 2
    rng = np.random.default_rng(H * 100 + W)
    x, rp, ci, va = synth.integer_case(N, C, H, W, K, m, r, 0.5, 300 + m)
    Ho, Wo = H + 2 * pad - r + 1, W + 2 * pad - r + 1
    G = rng.integers(-2, 3, size=(N, K, Ho, Wo)).astype(np.float32)
    print("case", H, W, m, r, pad, flush=True)
    ref = oracle.backward_f64(x, rp, ci, va, G, K, m, r, pad)[0]
    plan = sw.swconv_plan_create(N, C, H, W, K, m, r, pad)
    try:
        sw.swconv_set_weights(plan, rp, ci, va)
        xd, gd = torch.from_numpy(x).cuda(), torch.from_numpy(G).cuda()
        din = torch.full(x.shape, float("nan"), device="cuda")
        torch.cuda.synchronize()
        sw.swconv_backward(plan, torch.cuda.current_stream().cuda_stream, xd.data_ptr(), gd.data_ptr(), din.data_ptr(), 0)
        got = din.cpu().numpy().astype(np.float64)
    finally:
        sw.swconv_plan_destroy(plan)
    if r == 3:
        np.testing.assert_array_equal(got, ref)
    else:
        assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()


@pytest.mark.parametrize("H,W,pad", [(33, 31, 2), (17, 52, 0), (40, 4, 2), (54, 35, 2), (56, 56, 2), (64, 64, 0)])
@pytest.mark.parametrize("fuse", ["0", "2"])
def test_patches_of_5x5_filters_in_one_kernel_and_in_two(H, W, pad, fuse, monkeypatch):
    """F(4x4,5x5) by either route, whichever of them the plan would take: images of several passes of 64 tiles."""
    monkeypatch.setenv("SWCONV_FUSE_INPUT_GRAD", fuse)
    test_patches_meet(H, W, 4, 5, pad)


@pytest.mark.parametrize("N,C,H,W,one", [
    (1, 5, 27, 27, True),        # one pass of 64 tiles
    (1, 128, 32, 32, True),      # 64 tiles: still one
    (1, 128, 33, 32, False),     # two passes, 32 workgroups
    (24, 16, 40, 40, True),      # two passes, 96 workgroups
    (19, 17, 40, 40, False),     # ... and 95
    (48, 16, 64, 64, True),      # four passes, 192
    (16, 44, 64, 64, False),     # ... and 176
    (3, 256, 88, 88, True),      # eight passes: 192 are enough
    (1, 16, 96, 96, False),
])
def test_route_of_5x5_filters(N, C, H, W, one):
    K, P = 4, 64
    rp, ci, va = synth.bernoulli_weights(P, K, C, 0.05, 1)
    x, out = torch.zeros((N, C, H, W), device="cuda"), torch.zeros((N, K, H, W), device="cuda")
    din = torch.empty_like(x)
    plan = sw.swconv_plan_create(N, C, H, W, K, 4, 5, 2)
    try:
        sw.swconv_set_weights(plan, rp, ci, va)
        ms = sw.swconv_profile_backward(plan, 0, x.data_ptr(), out.data_ptr(), din.data_ptr(), 0, 1)
        assert ms[5] > 0 and (ms[6] == 0) == one
    finally:
        sw.swconv_plan_destroy(plan)
