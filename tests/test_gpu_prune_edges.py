"""The pruning step at the edges of its kernels, bit for bit against the oracle: rows of 15, 16, 17, 32 and 33 entries (16
lanes share a row), row counts around one round of the scan (16 x 1024) and around a run of 64; and more rows
than one launch has 16 lanes for."""
import numpy as np
import pytest
import torch

import oracle
from paper_1702_08597_amd import binding as sw
from test_gpu_prune_parity import gpu_prune

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 15, 17, 63, 65, 1025, 16383, 16384, 16385, 32769])
def test_prune_step_at_row_count_and_row_length_edges(rows):
    rng = np.random.default_rng(rows)
    lens = rng.choice([0, 1, 15, 16, 17, 32, 33], size=rows)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate([np.arange(n) for n in lens] + [np.zeros(0)]).astype(np.int32)
    va = (rng.standard_normal(rp[-1]) * 2e-3).astype(np.float32)
    g = (rng.standard_normal(rp[-1]) * 0.05).astype(np.float32)
    args = (0.01, 1e-3, 1e-4, 0.1)
    upd_o, (rp_o, ci_o, va_o) = oracle.prune_step(rp, ci, va, g, *args, np.float32)
    upd, rp2, ci2, va2, _ = gpu_prune(rp, ci, va, g, *args)
    np.testing.assert_array_equal(upd.view(np.uint32), upd_o.view(np.uint32))
    np.testing.assert_array_equal(rp2, rp_o)
    np.testing.assert_array_equal(ci2, ci_o)
    np.testing.assert_array_equal(va2.view(np.uint32), va_o.view(np.uint32))


def test_prune_step_on_more_rows_than_one_launch_covers():
    rows = (1 << 28) + 37
    rng = np.random.default_rng(28)
    # entries in the first rows, where the workgroups take their second turn (2^23 x 16 rows) and in the last rows
    full = np.concatenate([np.arange(40), np.arange((1 << 27) - 20, (1 << 27) + 20), np.arange(rows - 40, rows)])
    lens = rng.integers(0, 34, size=len(full))
    ci = np.concatenate([np.arange(n) for n in lens]).astype(np.int32)
    va = (rng.standard_normal(len(ci)) * 2e-3).astype(np.float32)
    g = (rng.standard_normal(len(ci)) * 0.05).astype(np.float32)
    args = (0.01, 1e-3, 1e-4, 0.1)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    upd_o, (rp_o, ci_o, va_o) = oracle.prune_step(rp, ci, va, g, *args, np.float32)

    def all_rows(rowptr):  # the row pointers with the empty rows in between
        count = torch.zeros(rows + 1, dtype=torch.int32, device="cuda")
        count[torch.from_numpy(full + 1).cuda()] = torch.from_numpy(np.diff(rowptr).astype(np.int32)).cuda()
        return torch.cumsum(count, 0, dtype=torch.int32)

    d = lambda a: torch.from_numpy(a).cuda()
    rpd, cid, vad, gd = all_rows(rp), d(ci), d(va), d(g)
    upd, va2 = torch.full_like(vad, float("nan")), torch.full_like(vad, float("nan"))
    rp2, ci2 = torch.full_like(rpd, -7), torch.full_like(cid, -7)
    sw.swconv_prune_step(rows, rpd.data_ptr(), cid.data_ptr(), vad.data_ptr(), gd.data_ptr(), *args,
                         torch.cuda.current_stream().cuda_stream, upd.data_ptr(), rp2.data_ptr(), ci2.data_ptr(),
                         va2.data_ptr())
    assert torch.equal(rp2, all_rows(rp_o))
    np.testing.assert_array_equal(upd.cpu().numpy().view(np.uint32), upd_o.view(np.uint32))
    np.testing.assert_array_equal(ci2.cpu().numpy()[:rp_o[-1]], ci_o)
    np.testing.assert_array_equal(va2.cpu().numpy()[:rp_o[-1]].view(np.uint32), va_o.view(np.uint32))
