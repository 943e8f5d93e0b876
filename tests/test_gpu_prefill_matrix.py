"""The 32x32 prefill kernel at the edges of what it walks: super-blocks of 32 token slots, groups of 64, workgroups of up
to 128 query rows, and a last block that is open at every fill, against the dense oracle (`assert_close`'s bounds)."""
import numpy as np
import pytest

import paper_2401_06761_amd as ap
from apar_workloads import HeadConfig, manual_tree, quantise
from oracle import DenseThreads

from harness import assert_close, blocks_upper_bound, pool_for, replay_trace, to_dev, to_host

pytestmark = pytest.mark.gpu

# (parents, segment lengths): each leaf's own segment is attended
SHAPES = {
    "every_fill": ([-1] * 17, list(range(1, 18))),
    "super_block_edges": ([-1] * 6, [31, 32, 33, 63, 64, 65]),
    "workgroup_edges": ([-1, 0, 0, 0, 0, 0], [49, 127, 128, 129, 160, 257]),
    "short_segments_on_long_paths": ([-1, 0, 0, 0, 0, 0, -1, 6, 6], [208, 1, 31, 33, 64, 96, 511, 17, 65]),
}


@pytest.mark.parametrize("n_q,n_kv", [(2, 2), (8, 2), (16, 1)])
@pytest.mark.parametrize("dtype", ["bf16", "bf16_fp8kv"])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_edges_of_the_walk(shape, dtype, n_q, n_kv):
    import torch

    parents, lens = SHAPES[shape]
    w = manual_tree(parents, lens, HeadConfig(n_q, n_kv, 128, dtype), seed=11)
    dense = DenseThreads(n_q, n_kv, 128)
    with pool_for(w, blocks_upper_bound(w)) as pool:
        pool.kv.fill_(0xFF)
        live, nodes = replay_trace(w, pool, None, dense)
        if dtype == "bf16":
            ap.apar_set_prefill_kernel(pool.handle, ap.APAR_PREFILL_MATRIX)
        rng = np.random.default_rng(2)
        for m in ([lens[i] for i in nodes], [dense.length(t) for t in live]):
            q = quantise(rng.standard_normal((sum(m), n_q, 128)).astype(np.float32), dtype)
            out = torch.full_like(to_dev(q, dtype), 3.0)
            ap.apar_prefill_attention(pool.handle, to_dev(q, dtype), live, m, out)
            torch.cuda.synchronize()
            if dtype == "bf16":
                assert ap.apar_last_prefill_kernel(pool.handle) == ap.APAR_PREFILL_MATRIX
            assert_close(to_host(out), dense.prefill(q, live, m), dtype, f"{sum(m)} query tokens")
