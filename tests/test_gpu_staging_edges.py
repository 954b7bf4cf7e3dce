"""The rows of a tile block go to LDS in dwords where a part of an image is short and in quads where it is longer than 256
floats, one to many images to a block; a span's last one to three floats travel by themselves.  Widths and heights
around that line and around whole quads and whole rounds of loads; odd planes put the channels on every alignment.
Tolerance: dL/dZ and the gradients against the oracle, the contract of the other backward tests, 1e-4 of the largest
value for F(4x4,3x3), 1e-5 for F(2x2,3x3)."""
import numpy as np
import pytest
import torch

from paper_1702_08597_amd import binding as sw
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


@pytest.mark.parametrize("H,W", [(16, 16), (17, 15), (16, 17), (8, 32), (8, 33)])
@pytest.mark.parametrize("m", [2, 4])
def test_staged_rows_around_the_line(H, W, m):
    test_staged_rows_of_every_length(H, W, m)


@pytest.mark.parametrize("H,W,m,r", [(13, 13, 4, 3), (56, 56, 4, 3), (30, 22, 2, 3), (24, 28, 4, 5), (32, 32, 2, 5)])
def test_tensors_that_start_at_any_float(H, W, m, r):
    """16-byte loads and stores of tensors that are aligned to 4 bytes: the bits of the aligned call, and nothing written
    beside the tensors."""
    N, C, K, P, pad = 3, 6, 8, (m + r - 1) ** 2, r // 2
    rp, ci, va = synth.bernoulli_weights(P, K, C, 0.4, 61)
    gen = torch.Generator(device="cuda").manual_seed(62)
    x, g = (torch.randn((N, c, H, W), generator=gen, device="cuda") for c in (C, K))
    plan = sw.swconv_plan_create(N, C, H, W, K, m, r, pad)
    try:
        sw.swconv_set_weights(plan, rp, ci, va)
        results = []
        for shift in (0, 1, 2, 3):
            def at(t):  # a copy of t that starts `shift` floats behind a 16-byte boundary, between guards
                flat = torch.full((t.numel() + 64,), 7.0, device="cuda")
                flat[32 + shift:32 + shift + t.numel()] = t.flatten()
                return flat
            xs, gs, out, din = at(x), at(g), at(torch.full_like(g, 7.0)), at(torch.full_like(x, 7.0))
            dv = torch.full((len(va) + 64,), 7.0, device="cuda")
            ptr = lambda flat: flat.data_ptr() + 4 * (32 + shift)
            sw.swconv_forward(plan, 0, ptr(xs), ptr(out))
            sw.swconv_backward(plan, 0, 0, ptr(gs), ptr(din), ptr(dv))
            torch.cuda.synchronize()
            res = []
            for flat, n in ((out, g.numel()), (din, x.numel()), (dv, len(va))):
                assert bool((flat[:32 + shift] == 7.0).all()) and bool((flat[32 + shift + n:] == 7.0).all())
                res.append(flat[32 + shift:32 + shift + n].clone())
            results.append(res)
        for res in results[1:]:
            for a, b in zip(res, results[0]):
                assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    finally:
        sw.swconv_plan_destroy(plan)
