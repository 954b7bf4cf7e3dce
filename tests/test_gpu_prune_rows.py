"""Row counts around the workgroups (16 rows) and turns (256 workgroups) of the pruning step without a scan, and around
the most rows it is used for (32768), and a power of two behind, each three times: which workgroups find their predecessors' entries already put
right differs from run to run, the result does not.  Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
from test_gpu_prune_parity import gpu_prune

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 16, 17, 32, 4095, 4096, 4097, 8193, 32767, 32768, 32769, 65535, 65536, 65537])
def test_row_pointers_without_a_scan(rows):
    rng = np.random.default_rng(rows)
    lens = rng.choice([0, 1, 5, 16, 17], size=rows)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate([np.arange(n) for n in lens] + [np.zeros(0)]).astype(np.int32)
    va = (rng.standard_normal(rp[-1]) * 2e-3).astype(np.float32)
    g = (rng.standard_normal(rp[-1]) * 0.05).astype(np.float32)
    args = (0.01, 1e-3, 1e-4, 0.1)
    upd_o, (rp_o, ci_o, va_o) = oracle.prune_step(rp, ci, va, g, *args, np.float32)
    for _ in range(3):
        upd, rp2, ci2, va2, _ = gpu_prune(rp, ci, va, g, *args)
        np.testing.assert_array_equal(upd.view(np.uint32), upd_o.view(np.uint32))
        np.testing.assert_array_equal(rp2, rp_o)
        np.testing.assert_array_equal(ci2, ci_o)
        np.testing.assert_array_equal(va2.view(np.uint32), va_o.view(np.uint32))
