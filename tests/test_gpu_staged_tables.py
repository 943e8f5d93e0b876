"""Tables of calls that are too large for the kernels' arguments: copied out of pinned memory by a kernel, and rewritten in
place by the calls that carry a plan over - on one stream and on two by turns."""
import numpy as np
import pytest

import paper_2401_06761_amd as ap
from apar_workloads import HeadConfig, manual_tree, quantise, step_q
from oracle import DenseThreads

from harness import assert_close, blocks_upper_bound, pool_for, replay_trace, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("requests", [1, 24, 150])  # plans of 1 KB (with the arguments), some 12 KB and 60 KB
@pytest.mark.parametrize("streams", [1, 2])
def test_decode_loop(dtype, d, requests, streams):
    import torch

    parents, lens = [], []
    for r in range(requests):
        parents += [-1] + [len(parents)] * 3
        lens += [20 + 7 * (r % 13), 1 + r % 17, 14, 40]
    w = manual_tree(parents, lens, HeadConfig(4, 2, d, dtype), seed=6)
    dense = DenseThreads(4, 2, d)
    with pool_for(w, blocks_upper_bound(w) + 6 * requests) as pool:
        pool.kv.fill_(0xFF)
        h = pool.handle
        live, _ = replay_trace(w, pool, None, dense)
        side = [torch.cuda.Stream() for _ in range(streams)]
        rng = np.random.default_rng(8)
        n = len(live)
        for step in range(4):
            k, v = (quantise(rng.standard_normal((n, 2, d)).astype(np.float32), dtype) for _ in range(2))
            ap.apar_append_kv_batch(h, live, to_dev(k, dtype), to_dev(v, dtype))
            for i, t in enumerate(live):
                dense.append(t, k[i:i + 1], v[i:i + 1])
            q = step_q(w, step, n)
            qd = to_dev(q, dtype)
            outs = [torch.full_like(qd, 3.0) for _ in range(3)]
            torch.cuda.synchronize()
            for i, out in enumerate(outs):
                side[i % streams].wait_stream(side[(i - 1) % streams])  # (the caller orders its streams)
                with torch.cuda.stream(side[i % streams]):
                    ap.apar_decode_attention(h, qd, live, out)
            torch.cuda.synchronize()
            assert_close(to_host(outs[0]), dense.decode(q, live), dtype, f"step {step}")
            assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
        assert ap.apar_plan_counts(h)[1] >= 8
