"""The input gradient of 3x3 filters by either route (one kernel that holds whole planes; patches, then a gather), bit for
bit against the oracle on integer data, on images of several passes of 64 tiles; and which of them a plan takes by passes
and workgroups."""
import pytest

from paper_1702_08597_amd import binding as sw
from paper_1702_08597_amd import synth
from test_gpu_input_grad_edges import test_patches_meet as patches_meet

import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,m,pad", [(33, 31, 2, 1), (17, 52, 2, 0), (56, 56, 2, 2), (54, 35, 4, 1), (40, 66, 4, 2),
                                       (64, 64, 4, 0)])
@pytest.mark.parametrize("fuse", ["0", "2"])
def test_patches_of_3x3_filters_in_one_kernel_and_in_two(H, W, m, pad, fuse, monkeypatch):
    monkeypatch.setenv("SWCONV_FUSE_INPUT_GRAD", fuse)
    patches_meet(H, W, m, 3, pad)


@pytest.mark.parametrize("N,C,H,m,one", [
    (1, 4, 32, 2, True),       # 4 passes
    (1, 252, 34, 2, False),    # 5 passes, 63 workgroups
    (1, 253, 34, 2, True),     # ... and 64
    (1, 256, 56, 2, False),    # 13 passes: 65 are needed
    (1, 4, 52, 4, True),       # 3 passes
    (4, 60, 56, 4, False),     # 4 passes, 60 workgroups
    (4, 64, 56, 4, True),      # ... and 64
])
def test_route_of_3x3_filters(N, C, H, m, one):
    K = 4
    rp, ci, va = synth.bernoulli_weights((m + 2) ** 2, K, C, 0.05, 1)
    x, out = torch.zeros((N, C, H, H), device="cuda"), torch.zeros((N, K, H, H), device="cuda")
    din = torch.empty_like(x)
    plan = sw.swconv_plan_create(N, C, H, H, K, m, 3, 1)
    try:
        sw.swconv_set_weights(plan, rp, ci, va)
        ms = sw.swconv_profile_backward(plan, 0, x.data_ptr(), out.data_ptr(), din.data_ptr(), 0, 1)
        assert ms[5] > 0 and (ms[6] == 0) == one
    finally:
        sw.swconv_plan_destroy(plan)
