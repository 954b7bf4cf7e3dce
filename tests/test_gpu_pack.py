"""The packing on the device (swconv_set_weights_device, and the transpose of W_F for the backward pass) against the
host's packing of the same arrays: exported weights, passes in both directions and the statistics have to be equal bit
for bit, the schedule a partition.  Sizes at the edges of its workgroups: one row, rows that fill no slice, more than
1024 and the most rows a workgroup sorts (4096), the first size beyond (which goes through the host), several column
checks per position, one and 638 columns (rows of up to 638 entries, 20 words of the transpose's bit matrix), empty,
full and skewed patterns."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1702_08597_amd import binding as sw
from paper_1702_08597_amd import synth

pytestmark = pytest.mark.gpu


def set_device(plan, rp, ci, va):
    dev = [torch.from_numpy(a).cuda() if len(a) else None for a in (rp, ci, va)]
    st = torch.cuda.current_stream().cuda_stream
    return sw.lib().swconv_set_weights_device(plan, ctypes.c_void_p(st),
                                              *(ctypes.c_void_p(a.data_ptr()) if a is not None else None for a in dev))


def passes(plan, x, g, K, nnz, backward):
    N, C, H, W = x.shape
    P, T, Ho, Wo = sw.swconv_plan_sizes(plan)
    out = torch.full((N, K, Ho, Wo), float("nan"), device="cuda")
    din = torch.full(x.shape, float("nan"), device="cuda")
    dv = torch.full((max(1, nnz),), float("nan"), device="cuda")
    sw.swconv_forward(plan, 0, x.data_ptr(), out.data_ptr())
    if backward:
        sw.swconv_backward(plan, 0, 0, g.data_ptr(), din.data_ptr(), dv.data_ptr())
    torch.cuda.synchronize()
    res = [out.cpu().numpy()] + ([din.cpu().numpy(), dv.cpu().numpy()[:nnz]] if backward else [])
    assert not any(np.isnan(r).any() for r in res)
    return res


@pytest.mark.parametrize("N,C,K,m,r,H,W,density,skew", [
    (1, 1, 1, 2, 3, 3, 3, 1.0, False),
    (2, 5, 7, 4, 3, 9, 6, 0.5, False),
    (3, 33, 127, 4, 3, 13, 13, 0.1, False),
    (2, 64, 129, 2, 5, 11, 7, 0.1, False),    # the fused format as well, two column checks per position
    (1, 24, 70, 4, 5, 9, 9, 0.0, False),
    (2, 48, 128, 2, 5, 27, 27, 0.094, False),
    (4, 96, 384, 4, 3, 13, 13, 0.1, True),
    (1, 638, 9, 2, 3, 6, 6, 1.0, False),
    (1, 20, 638, 2, 3, 6, 6, 0.3, False),
    (1, 3, 1030, 2, 3, 6, 6, 0.7, False),     # more rows than threads; K beyond the backward pass
    (1, 2, 4096, 2, 3, 6, 6, 0.6, False),
    (1, 2, 4097, 2, 3, 6, 6, 0.6, False),     # through the host
])
def test_device_packing_equals_host_packing(N, C, K, m, r, H, W, density, skew):
    P = (m + r - 1) ** 2
    rp, ci, va = synth.skewed_weights(P, K, C, 5 + K) if skew else synth.bernoulli_weights(P, K, C, density, 5 + K)
    x = torch.from_numpy(synth.activations(N, C, H, W, 6)).cuda()
    plans = [sw.swconv_plan_create(N, C, H, W, K, m, r, r // 2) for _ in range(2)]
    try:
        sw.swconv_set_weights(plans[0], rp, ci, va)
        # another pattern first, so that the call really replaces weights (and shrinks or grows every buffer)
        rp0, ci0, va0 = synth.bernoulli_weights(P, K, C, 0.25, 7)
        assert set_device(plans[1], rp0, ci0, va0) == sw.SWCONV_OK
        assert set_device(plans[1], rp, ci, va) == sw.SWCONV_OK
        rp2, ci2, va2 = sw.swconv_debug_export_weights(plans[1], K, len(va))
        np.testing.assert_array_equal(rp2, rp)
        np.testing.assert_array_equal(ci2, ci)
        np.testing.assert_array_equal(va2.view(np.uint32), va.view(np.uint32))
        sw.swconv_debug_check_schedule(plans[1])
        a, b = (sw.swconv_plan_weight_stats(p) for p in plans)
        assert (a["nnz"], a["padded_nnz"]) == (b["nnz"], b["padded_nnz"])
        Ho, Wo = sw.swconv_plan_sizes(plans[0])[2:]
        g = torch.randn((N, K, Ho, Wo), generator=torch.Generator(device="cuda").manual_seed(8), device="cuda")
        for p, q in zip(*(passes(pl, x, g, K, len(va), K <= 638) for pl in plans)):
            np.testing.assert_array_equal(p.view(np.uint32), q.view(np.uint32))
        for pl in plans:
            sw.swconv_debug_check_schedule(pl)  # now the transpose's too
    finally:
        for pl in plans:
            sw.swconv_plan_destroy(pl)


def test_schedule_of_a_pattern_that_stays_is_the_hosts():
    """A plan's first pattern, and one that replaces a pattern of 512 passes, get the schedule that swconv_set_weights
    makes; the patterns of a loop get the device's.  The results are the same."""
    N, K, C = 32, 96, 64
    rp, ci, va = synth.bernoulli_weights(36, K, C, 0.1, 21)
    x = torch.from_numpy(synth.activations(N, C, 13, 13, 22)).cuda()
    g = torch.randn((N, K, 13, 13), generator=torch.Generator(device="cuda").manual_seed(23), device="cuda")
    host, dev = (sw.swconv_plan_create(N, C, 13, 13, K, 4, 3, 1) for _ in range(2))
    try:
        sw.swconv_set_weights(host, rp, ci, va)
        want, stats = passes(host, x, g, K, len(va), True), sw.swconv_plan_weight_stats(host)
        for turn, even in enumerate((True, False, True)):
            assert set_device(dev, rp, ci, va) == sw.SWCONV_OK
            assert (sw.swconv_plan_weight_stats(dev) == stats) == even, turn
            for a, b in zip(passes(dev, x, g, K, len(va), True), want):
                np.testing.assert_array_equal(a.view(np.uint32), b.view(np.uint32))
            sw.swconv_debug_check_schedule(dev)
            if turn == 1:
                out = torch.empty_like(g)
                for _ in range(510):  # with the forward and the backward pass above: 512
                    sw.swconv_forward(dev, 0, x.data_ptr(), out.data_ptr())
    finally:
        for p in (host, dev):
            sw.swconv_plan_destroy(p)


@pytest.mark.parametrize("from_device", [False, True])
def test_backward_buffers_are_sized_by_the_batches_there_are(from_device):
    """The partial sums of dL/dW_F: one float per tile block and pair of the transpose's batches, of which a slice of
    four rows has ceil(longest / 16).  No more of them are held than there are."""
    N, C, H, W, K, m, r = 256, 48, 27, 27, 128, 4, 5
    rp, ci, va = synth.bernoulli_weights(64, K, C, 0.094, 31)
    batches = 0
    for p in range(64):
        lens = np.bincount(ci[rp[p * K]:rp[(p + 1) * K]], minlength=C)
        batches += int(np.ceil(np.sort(lens)[::-1][::4] / 16).sum())
    x, out = torch.zeros((N, C, H, W), device="cuda"), torch.zeros((N, K, H, W), device="cuda")
    din, dv = torch.empty_like(x), torch.empty(len(va), device="cuda")
    plan = sw.swconv_plan_create(N, C, H, W, K, m, r, 2)
    try:
        if from_device:
            assert set_device(plan, rp, ci, va) == sw.SWCONV_OK
        else:
            sw.swconv_set_weights(plan, rp, ci, va)
        sw.swconv_forward(plan, 0, x.data_ptr(), out.data_ptr())
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        sw.swconv_backward(plan, 0, 0, out.data_ptr(), din.data_ptr(), dv.data_ptr())
        torch.cuda.synchronize()
        held = before - torch.cuda.mem_get_info()[0]
        tiles = -(-sw.swconv_plan_sizes(plan)[1] // 128) * 128
        gradient, partial = 64 * C * tiles * 4, tiles // 64 * (batches + 2) * 64 * 4
        assert gradient + partial <= held <= gradient + partial + (24 << 20)  # and the packed weights, tables, rounding
    finally:
        sw.swconv_plan_destroy(plan)


@pytest.mark.parametrize("N,C,H,W,K,m,r,density,fuse", [
    (3, 48, 27, 27, 128, 2, 5, 0.094, None),  # the fused product + output transform: one batch per slice, two at most
    (2, 40, 13, 13, 70, 2, 3, 0.3, None),     # ... rows of up to 32 entries, a broken chunk of 64 rows
    (2, 64, 13, 13, 96, 4, 3, 0.1, "2"),      # the fused kernel of F(4x4,3x3), where asked for: whole units of two batches
    (1, 200, 13, 13, 65, 4, 3, 0.55, "2"),    # ... rows of more than 96 entries, one row in the last chunk
    (2, 64, 13, 13, 96, 4, 3, 0.1, None),
])
def test_values_updated_in_a_device_packed_plan(N, C, H, W, K, m, r, density, fuse, monkeypatch):
    """swconv_update_values goes through the index that the packing wrote with every packed copy - stream, transpose and,
    where steps 2 and 3 run fused, packages: the same bits as a plan given the new values by the host."""
    if fuse:
        monkeypatch.setenv("SWCONV_FUSE_OUTPUT", fuse)
    P = (m + r - 1) ** 2
    rp, ci, va = synth.bernoulli_weights(P, K, C, density, 41)
    new = np.random.default_rng(42).standard_normal(len(va)).astype(np.float32)
    x = torch.from_numpy(synth.activations(N, C, H, W, 43)).cuda()
    plans = [sw.swconv_plan_create(N, C, H, W, K, m, r, r // 2) for _ in range(2)]
    try:
        Ho, Wo = sw.swconv_plan_sizes(plans[0])[2:]
        g = torch.randn((N, K, Ho, Wo), generator=torch.Generator(device="cuda").manual_seed(44), device="cuda")
        sw.swconv_set_weights(plans[0], rp, ci, new)
        assert set_device(plans[1], rp, ci, va) == sw.SWCONV_OK
        out, fused = torch.empty_like(g), fuse is not None or m == 2
        ms = sw.swconv_profile_forward(plans[1], 0, x.data_ptr(), out.data_ptr(), 1)
        assert (ms[2] == 0) == fused  # the route that the case is here for
        for before_backward in (True, False):  # the transpose is packed by the first backward pass
            values = torch.from_numpy(new if not before_backward else -new).cuda()
            sw.swconv_update_values(plans[1], 0, values.data_ptr())
            got = passes(plans[1], x, g, K, len(va), True)
        for a, b in zip(got, passes(plans[0], x, g, K, len(va), True)):
            np.testing.assert_array_equal(a.view(np.uint32), b.view(np.uint32))
    finally:
        for pl in plans:
            sw.swconv_plan_destroy(pl)


@pytest.mark.parametrize("N,C,H,W,K,density", [(32, 64, 27, 27, 96, 0.1), (24, 96, 30, 26, 100, 0.05)])
def test_device_cut_of_a_transpose_with_two_workgroups_per_cu(N, C, H, W, K, density):
    """More than 32 units per compute unit: both operands run two workgroups on each, by the device's cut."""
    rp, ci, va = synth.bernoulli_weights(36, K, C, density, 51)
    x = torch.from_numpy(synth.activations(N, C, H, W, 52)).cuda()
    g = torch.randn((N, K, H, W), generator=torch.Generator(device="cuda").manual_seed(53), device="cuda")
    plans = [sw.swconv_plan_create(N, C, H, W, K, 4, 3, 1) for _ in range(2)]
    try:
        tiles = sw.swconv_plan_sizes(plans[0])[1]
        assert 36 * -(-tiles // 64) * (C // 4) >= 32 * torch.cuda.get_device_properties(0).multi_processor_count
        sw.swconv_set_weights(plans[0], rp, ci, va)
        for _ in range(2):  # the second one is a loop's: the device cuts
            assert set_device(plans[1], rp, ci, va) == sw.SWCONV_OK
        for a, b in zip(*(passes(pl, x, g, K, len(va), True) for pl in plans)):
            np.testing.assert_array_equal(a.view(np.uint32), b.view(np.uint32))
        for pl in plans:
            sw.swconv_debug_check_schedule(pl)
    finally:
        for pl in plans:
            sw.swconv_plan_destroy(pl)


def test_queries_of_a_device_packed_plan_read_the_plan_and_nothing_else():
    K, C = 96, 64
    rp, ci, va = synth.bernoulli_weights(36, K, C, 0.1, 9)
    plan = sw.swconv_plan_create(2, C, 13, 13, K, 4, 3, 1)
    x, out = torch.randn((2, C, 13, 13), device="cuda"), torch.zeros((2, K, 13, 13), device="cuda")
    try:
        assert set_device(plan, rp, ci, va) == sw.SWCONV_OK
        sw.swconv_forward(plan, torch.cuda.current_stream().cuda_stream, x.data_ptr(), out.data_ptr())
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):  # a call that waited for the device here would end the capture
            sw.swconv_forward(plan, torch.cuda.current_stream().cuda_stream, x.data_ptr(), out.data_ptr())
            during = sw.swconv_plan_weight_stats(plan)
        sw.swconv_debug_check_schedule(plan)  # the statistics against the schedule that the device holds
        assert during == sw.swconv_plan_weight_stats(plan)
        assert during["nnz"] == len(va) and during["work_items"] > 0 and during["max_item"] > 0
        want = out.clone()
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    finally:
        sw.swconv_plan_destroy(plan)


def test_packing_is_refused_under_capture():
    """A packing that a capture only records has not happened, whatever the plan then notes: the first backward pass
    on new weights and the new weights themselves are refused there, and the eager passes after it are right."""
    N, K, C = 2, 96, 64
    patterns = [synth.bernoulli_weights(36, K, C, d, 11) for d in (0.2, 0.1)]
    x = torch.from_numpy(synth.activations(N, C, 13, 13, 12)).cuda()
    g = torch.randn((N, K, 13, 13), generator=torch.Generator(device="cuda").manual_seed(13), device="cuda")
    plan, fresh = (sw.swconv_plan_create(N, C, 13, 13, K, 4, 3, 1) for _ in range(2))
    try:
        assert set_device(plan, *patterns[0]) == sw.SWCONV_OK
        passes(plan, x, g, K, len(patterns[0][2]), True)  # every buffer there is, larger than the second pattern needs
        assert set_device(plan, *patterns[1]) == sw.SWCONV_OK
        arrays = [torch.from_numpy(a).cuda() for a in patterns[1]]
        out, din, dv = torch.empty_like(g), torch.empty_like(x), torch.empty(len(patterns[1][2]), device="cuda")
        ptr = lambda t: ctypes.c_void_p(t.data_ptr())
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            st = torch.cuda.current_stream().cuda_stream
            sw.swconv_forward(plan, st, x.data_ptr(), out.data_ptr())
            status = [sw.lib().swconv_backward(plan, ctypes.c_void_p(st), ptr(x), ptr(g), ptr(din), ptr(dv)),
                      sw.lib().swconv_set_weights_device(plan, ctypes.c_void_p(st), *(ptr(a) for a in arrays))]
        assert status == [sw.SWCONV_EHIP, sw.SWCONV_EHIP]
        sw.swconv_set_weights(fresh, *patterns[1])
        for a, b in zip(*(passes(p, x, g, K, len(patterns[1][2]), True) for p in (plan, fresh))):
            np.testing.assert_array_equal(a.view(np.uint32), b.view(np.uint32))
    finally:
        for p in (plan, fresh):
            sw.swconv_plan_destroy(p)


def test_malformed_device_arrays_are_refused_and_the_weights_stay():
    K, C = 130, 40
    rp, ci, va = synth.bernoulli_weights(36, K, C, 0.3, 3)
    plan = sw.swconv_plan_create(2, C, 13, 13, K, 4, 3, 1)
    try:
        assert set_device(plan, rp, ci, va) == sw.SWCONV_OK
        last = int(rp[-2])  # first entry of the last row, which the second column check of its position reads
        full = next(i for i in range(36 * K) if rp[i + 1] - rp[i] >= 2)

        def bad(a, where, value):
            b = a.copy()
            b[where] = value
            return b

        for args in ((bad(rp, 0, 1), ci, va), (bad(rp, 5, rp[4] - 1), ci, va), (bad(rp, 7, rp[-1] + 1), ci, va),
                     (bad(rp, 9, -3), ci, va), (bad(rp, -1, -1), ci, va), (rp, bad(ci, last, C), va),
                     (rp, bad(ci, rp[full], -1), va), (rp, bad(ci, rp[full] + 1, ci[rp[full]]), va),
                     (bad(rp, slice(1, 3), rp[3] + C), ci, va)):
            assert set_device(plan, *args) == sw.SWCONV_EINVAL
        assert sw.lib().swconv_set_weights_device(plan, None, None, None, None) == sw.SWCONV_EINVAL
        d = torch.from_numpy(rp).cuda()
        assert sw.lib().swconv_set_weights_device(plan, None, ctypes.c_void_p(d.data_ptr()), None, None) == sw.SWCONV_EINVAL
        rp2, ci2, va2 = sw.swconv_debug_export_weights(plan, K, len(va))
        np.testing.assert_array_equal(rp2, rp)
        np.testing.assert_array_equal(ci2, ci)
        np.testing.assert_array_equal(va2, va)
    finally:
        sw.swconv_plan_destroy(plan)
