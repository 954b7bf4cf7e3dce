"""The inner loops of the sparse product where they can go wrong: slices of every number of steps (units of two batches,
their exits after each group of four steps, slices of none, one and several units), plans with and without slices of more
than 32 steps, every size of panel a workgroup stages, items that are ragged (few rows, one tile, several tile blocks),
plans whose rows pass 32 entries and come back, and weights the broadcast has to carry (denormal, huge, infinite, NaN).

Integer data: M and the backward pass's D and dvals equal to the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_1702_08597_amd import binding as sw

pytestmark = pytest.mark.gpu


def rows_of_lengths(P, K, C, lengths, rng):
    """Per-position CSR whose row (p, k) holds lengths(p, k) entries, at most C, in random columns."""
    rp, ci = [0], []
    for p in range(P):
        for k in range(K):
            ci.append(np.sort(rng.permutation(C)[:min(C, lengths(p, k))]))
            rp.append(rp[-1] + len(ci[-1]))
    ci = np.concatenate(ci).astype(np.int32)
    return np.array(rp, dtype=np.int32), ci, rng.integers(-2, 3, size=len(ci)).astype(np.float32)


def passes(N, C, H, W, K, m, rp, ci, va, x, G):
    plan = sw.swconv_plan_create(N, C, H, W, K, m, 3, 1)
    try:
        sw.swconv_set_weights(plan, rp, ci, va)
        assert sw.swconv_debug_check_schedule(plan) in (None, 0)
        xd, gd = torch.from_numpy(x).cuda(), torch.from_numpy(G).cuda()
        out, din = torch.empty((N, K, H, W), device="cuda"), torch.empty_like(xd)
        dvals = torch.full((max(1, len(va)),), float("nan"), device="cuda")
        torch.cuda.synchronize()
        sw.swconv_forward(plan, 0, xd.data_ptr(), out.data_ptr())
        M = sw.swconv_debug_copy_M(plan, K)
        sw.swconv_backward(plan, 0, 0, gd.data_ptr(), din.data_ptr(), dvals.data_ptr())
        torch.cuda.synchronize()
        return M, sw.swconv_debug_copy_dV(plan, C), dvals.cpu().numpy()[:len(va)]
    finally:
        sw.swconv_plan_destroy(plan)


# panels of one to seven pieces at 12 waves, six and ten at 16, and at the edges between them
@pytest.mark.parametrize("C,K", [(40, 24), (96, 64), (97, 50), (288, 40), (289, 37), (319, 21), (320, 64), (384, 96),
                                 (385, 33), (600, 19)])
@pytest.mark.parametrize("longest", [32, 33, 600])
def test_slices_of_every_length(C, K, longest):
    N, H, W, m, P = 5, 9, 11, 2, 16
    rng = np.random.default_rng(C + longest)
    # rows of 0, 1, 2, ... entries, each length in a slice of its own at some position
    rp, ci, va = rows_of_lengths(P, K, C, lambda p, k: (p * 7 + k * 5) % (min(longest, C) + 1), rng)
    x = rng.integers(0, 4, size=(N, C, H, W)).astype(np.float32)
    G = rng.integers(-2, 3, size=(N, K, H, W)).astype(np.float32)
    print("case", C, K, longest, flush=True)
    M, D, dvals = passes(N, C, H, W, K, m, rp, ci, va, x, G)
    M64 = oracle.forward_f64(x, rp, ci, va, K, m)[2]
    _, dvals64, _, D64 = oracle.backward_f64(x, rp, ci, va, G, K, m)
    np.testing.assert_array_equal(M.astype(np.float64), M64)
    np.testing.assert_array_equal(D.astype(np.float64), D64)
    np.testing.assert_array_equal(dvals.astype(np.float64), dvals64)


def products_of_single_entries(special, seed):
    """M and what numpy makes of it, for one entry a row: every product is one multiplication."""
    N, C, H, W, K, m, P = 2, 130, 6, 6, 22, 2, 16
    rng = np.random.default_rng(seed)
    rp, ci, va = rows_of_lengths(P, K, C, lambda p, k: 1, rng)
    va = np.array(special, np.float32)[rng.integers(0, len(special), size=len(va))]
    x = np.zeros((N, C, H, W), np.float32)
    x[:, :, ::2, ::2] = rng.integers(0, 2, size=(N, C, 3, 3))  # V holds small integers
    plan = sw.swconv_plan_create(N, C, H, W, K, m, 3, 1)
    try:
        sw.swconv_set_weights(plan, rp, ci, va)
        xd, out = torch.from_numpy(x).cuda(), torch.empty((N, K, H, W), device="cuda")
        sw.swconv_forward(plan, 0, xd.data_ptr(), out.data_ptr())
        V, M = sw.swconv_debug_copy_V(plan, C), sw.swconv_debug_copy_M(plan, K)
    finally:
        sw.swconv_plan_destroy(plan)
    col = ci.reshape(P, K)
    with np.errstate(over="ignore", invalid="ignore"):
        want = va.reshape(P, K, 1) * np.stack([V[p][col[p]] for p in range(P)]) + np.float32(0)
    assert M.dtype == want.dtype == np.float32
    return M, want


def test_weights_are_broadcast_unchanged():
    """The single float product, bit for bit.  (A weight of -0 comes out as +0, which no sum that starts at +0 shows.)"""
    M, want = products_of_single_entries([1e-45, -1e-45, 1.17e-38, -3.3e-39, 3.4e38, -3.4e38, -0.0, 1.0, -1.5, 2.0 ** -126], 3)
    np.testing.assert_array_equal(M.view(np.uint32), want.view(np.uint32))


def test_infinite_and_nan_weights_stay_in_their_rows():
    """Four rows share a slice, a matrix instruction and their registers."""
    M, want = products_of_single_entries([np.inf, -np.inf, np.nan, 1.0, -2.0, 0.5], 4)
    assert np.isnan(want).any() and np.isinf(want).any() and np.isfinite(want).any()
    np.testing.assert_array_equal(M, want)


@pytest.mark.parametrize("C,K", [(70, 40), (330, 24)])
def test_rows_pass_32_entries_and_come_back(C, K):
    """The product is built for rows of up to 32 entries and for longer ones: new patterns on the device move a plan from
    one to the other."""
    N, H, W, m, P = 5, 9, 11, 2, 16
    rng = np.random.default_rng(C)
    x = rng.integers(0, 4, size=(N, C, H, W)).astype(np.float32)
    xd, out = torch.from_numpy(x).cuda(), torch.empty((N, K, H, W), device="cuda")
    plan = sw.swconv_plan_create(N, C, H, W, K, m, 3, 1)
    try:
        for longest in (32, 33, 31, 65, 32, 1):
            print("case", C, K, longest, flush=True)
            rp, ci, va = rows_of_lengths(P, K, C, lambda p, k: (p * 7 + k * 5) % longest if (p, k) != (3, 2) else longest, rng)
            dev = [torch.from_numpy(a).cuda() for a in (rp, ci, va)]
            sw.swconv_set_weights_device(plan, 0, *(d.data_ptr() for d in dev))
            sw.swconv_debug_check_schedule(plan)
            sw.swconv_forward(plan, 0, xd.data_ptr(), out.data_ptr())
            M = sw.swconv_debug_copy_M(plan, K)
            ref, _, M64 = oracle.forward_f64(x, rp, ci, va, K, m)
            np.testing.assert_array_equal(M.astype(np.float64), M64)
            np.testing.assert_array_equal(out.cpu().numpy().astype(np.float64), ref)
    finally:
        sw.swconv_plan_destroy(plan)
