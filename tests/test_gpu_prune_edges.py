"""The pruning step at the edges of its kernels, bit for bit against the oracle: rows of 15, 16, 17, 32 and 33 entries (16
lanes share a row), row counts around one round of the scan (16 x 1024) and around a run of 64."""
import numpy as np
import pytest

import oracle
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
