"""Steps 2 and 3 of m = 2 layers in one kernel (rows of V gathered from memory, the positions of a slice on the waves of a
workgroup) against the three kernels - the same bits - and against the oracle: rows at the edges of the step groups and
batches, up to the longest the packages hold, broken slices and chunks of rows, tiles that end inside the output, tile
blocks that span images and are broken, one position or two to a wave, channel groups of larger tensors."""
import numpy as np
import pytest
import torch

import oracle
from paper_1702_08597_amd import binding as sw
from paper_1702_08597_amd import synth

pytestmark = pytest.mark.gpu
RTOL = {3: 1e-5, 5: 1e-4}


def forward(mode, monkeypatch, x, rp, ci, va, K, r, pad, group=None):
    """One pass; `group` = (channels of the whole input, of the whole output) places the layer inside larger tensors."""
    monkeypatch.setenv("SWCONV_FUSE_OUTPUT", mode)
    N, C, H, W = x.shape
    Ho, Wo = H + 2 * pad - r + 1, W + 2 * pad - r + 1
    plan = sw.swconv_plan_create(N, C, H, W, K, 2, r, pad)
    try:
        sw.swconv_set_weights(plan, rp, ci, va)
        Ca, Ka = group or (C, K)
        if group:
            sw.swconv_plan_set_image_strides(plan, Ca * H * W, Ka * Ho * Wo)
        xd = torch.zeros((N, Ca, H, W), device="cuda")
        xd[:, Ca - C:] = torch.from_numpy(x).cuda()
        out = torch.full((N, Ka, Ho, Wo), float("nan"), device="cuda")
        args = (plan, 0, xd.data_ptr() + 4 * (Ca - C) * H * W, out.data_ptr() + 4 * (Ka - K) * Ho * Wo)
        sw.swconv_forward(*args)
        ms = sw.swconv_profile_forward(*args, 1)
        assert torch.isnan(out[:, :Ka - K]).all()
        return out[:, Ka - K:].cpu().numpy(), ms[2] == 0
    finally:
        sw.swconv_plan_destroy(plan)


def csr(P, K, C, length, rng):
    rows = [np.sort(rng.permutation(C)[:length(p, k)]) for p in range(P) for k in range(K)]
    rp = np.concatenate([[0], np.cumsum([len(q) for q in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    return rp, ci, (rng.standard_normal(len(ci)) * 0.05).astype(np.float32)


@pytest.mark.parametrize("r", [3, 5])
@pytest.mark.parametrize("N,C,H,W,K,longest,one", [
    (1, 60, 7, 5, 1, 48, True),      # every length from none to 48, one row, one tile block
    (3, 64, 13, 13, 70, 16, True),   # a broken slice, two chunks of 64 rows, images that share a tile block
    (2, 70, 9, 12, 130, 17, True),   # two batches
    (2, 70, 9, 12, 131, 33, True),   # three
    (2, 70, 9, 12, 3, 49, False),    # longer than the packages hold: three kernels
    (7, 300, 10, 11, 259, 12, True),  # more workgroups than there are CUs
    (7, 70, 10, 11, 259, 17, True),   # ... and two batches
    (7, 70, 10, 11, 259, 33, True),   # ... and three
    (7, 70, 10, 11, 259, 48, True),
])
def test_equals_the_three_kernels(r, N, C, H, W, K, longest, one, monkeypatch):
    rng = np.random.default_rng(longest + r)
    P, pad = (r + 1) ** 2, r // 2
    rp, ci, va = csr(P, K, C, lambda p, k: longest if (p, k) == (P - 1, K - 1) else (p * 5 + k * 3) % (longest + 1), rng)
    x = synth.activations(N, C, H, W, 9)
    print("case", r, N, C, H, W, K, longest, flush=True)
    got, fused = forward("2", monkeypatch, x, rp, ci, va, K, r, pad)
    assert fused == one
    want, fused = forward("0", monkeypatch, x, rp, ci, va, K, r, pad)
    assert not fused
    np.testing.assert_array_equal(got.view(np.uint32), want.view(np.uint32))
    ref = oracle.forward_f64(x, rp, ci, va, K, 2, r, pad, want_VM=False)[0]
    assert np.abs(got - ref).max() <= RTOL[r] * np.abs(ref).max()


@pytest.mark.parametrize("r", [3, 5])
def test_inside_larger_tensors(r, monkeypatch):
    rng = np.random.default_rng(r)
    rp, ci, va = csr((r + 1) ** 2, 22, 24, lambda p, k: (p + k) % 9, rng)
    x = synth.activations(3, 24, 9, 10, 4)
    got, fused = forward("2", monkeypatch, x, rp, ci, va, 22, r, r // 2, (30, 25))
    assert fused
    want, _ = forward("0", monkeypatch, x, rp, ci, va, 22, r, r // 2)
    np.testing.assert_array_equal(got.view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("N,C,H,W,K,r,density,one", [
    (1, 256, 13, 13, 384, 3, 0.1, True),    # 38 MB of rows, M of 2 MB
    (4, 256, 13, 13, 384, 3, 0.1, False),   # 155 and 5: M is the smaller matter
    (32, 48, 27, 27, 128, 5, 0.094, True),  # 502 and 110
    (32, 64, 27, 27, 128, 3, 0.1, False),   # 317 and 49
])
def test_route_by_size(N, C, H, W, K, r, density, one, monkeypatch):
    rp, ci, va = synth.bernoulli_weights((r + 1) ** 2, K, C, density, 3)
    x = synth.activations(N, C, H, W, 5)
    assert forward("1", monkeypatch, x, rp, ci, va, K, r, r // 2)[1] == one


@pytest.mark.parametrize("N", [24, 56, 61, 62, 64])
def test_route_does_not_jump_with_the_batch(N, monkeypatch):
    """56 x 56, 32 -> 32 channels at 20 %: M passes 96 MB between 62 and 63 images; one kernel is the faster way for all."""
    rp, ci, va = synth.bernoulli_weights(16, 32, 32, 0.2, 3)
    x = np.zeros((N, 32, 56, 56), np.float32)
    assert forward("1", monkeypatch, x, rp, ci, va, 32, 3, 1)[1]
