"""fp8 pools on the 32x32 prefill kernel (taken by default from 32 query rows per thread on): sealed tiles widened as they
are staged, the walk's last block open or full, against the oracle and against the row-tile kernel."""
import numpy as np
import pytest

import paper_2401_06761_amd as ap
from apar_workloads import HeadConfig, manual_tree, quantise
from oracle import DenseThreads

from harness import assert_close, blocks_upper_bound, pool_for, replay_trace, to_dev, to_host

pytestmark = pytest.mark.gpu
F8 = "bf16_fp8kv"


@pytest.mark.parametrize("n_q,n_kv", [(2, 2), (8, 2), (16, 1)])
@pytest.mark.parametrize("lens", [[33, 7, 64, 16], [128, 1, 129, 63], [15, 300, 17, 33]])
def test_matrix_prefill_on_fp8_blocks(n_q, n_kv, lens):
    import torch

    w = manual_tree([-1, 0, 0, -1], lens, HeadConfig(n_q, n_kv, 128, F8), seed=9)
    dense = DenseThreads(n_q, n_kv, 128)
    with pool_for(w, blocks_upper_bound(w)) as pool:
        pool.kv.fill_(0xFF)
        live, _ = replay_trace(w, pool, None, dense)
        m = [dense.length(t) for t in live]
        rng = np.random.default_rng(4)
        q = quantise(rng.standard_normal((sum(m), n_q, 128)).astype(np.float32), F8)
        want = dense.prefill(q, live, m)
        for setting, kernel in ((ap.APAR_PREFILL_AUTO, None), (ap.APAR_PREFILL_ROW_TILES, ap.APAR_PREFILL_ROW_TILES)):
            ap.apar_set_prefill_kernel(pool.handle, setting)
            out = torch.empty_like(to_dev(q, F8))
            ap.apar_prefill_attention(pool.handle, to_dev(q, F8), live, m, out)
            torch.cuda.synchronize()
            if kernel is None:
                kernel = ap.APAR_PREFILL_MATRIX if sum(m) * (n_q // n_kv) >= 32 * len(live) else ap.APAR_PREFILL_ROW_TILES
            assert ap.apar_last_prefill_kernel(pool.handle) == kernel
            assert_close(to_host(out), want, F8, f"setting {setting}")
