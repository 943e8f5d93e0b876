"""Units cut into slices (calls with few threads): every slice count and list shape gives what the oracle gives, the
same call twice gives the same bits (the fold is in slice order and leaves its counters at zero), and the entry point
that allocates nothing cuts the same way."""
import numpy as np
import pytest

import paper_2401_06761_amd as ap
from apar_workloads import HeadConfig, draw_candidate_tree, manual_tree, mask_rows_from_parents, spec_step_qkv, step_q
from oracle import DenseThreads

from harness import assert_close, blocks_upper_bound, pool_for, replay_trace, to_dev, to_host

pytestmark = pytest.mark.gpu

# (parents, segment lengths): one long thread; a long root with short leaves; wide enough for two row tiles; packed
# short units beside a long one
SHAPES = {
    "one_thread": ([-1], [1613]),
    "one_block": ([-1, 0], [3, 9]),
    "long_root": ([-1, 0, 0, 0], [2100, 1, 17, 40]),
    "two_row_tiles": ([-1] + [0] * 70, [400] + [1 + 7 * (i % 9) for i in range(70)]),
    "uneven": ([-1, 0, 0, -1, -1, 4, 4, -1], [900, 300, 16, 5, 33, 2, 1, 16]),
}


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16_fp8kv", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("n_q,n_kv", [(2, 2), (8, 1), (5, 1)])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_slices_against_the_oracle(dtype, d, n_q, n_kv, shape):
    import torch

    parents, lens = SHAPES[shape]
    w = manual_tree(parents, lens, HeadConfig(n_q, n_kv, d, dtype), seed=3)
    dense = DenseThreads(n_q, n_kv, d)
    with pool_for(w, blocks_upper_bound(w)) as pool:
        pool.kv.fill_(0xFF)
        h = pool.handle
        live, _ = replay_trace(w, pool, None, dense)
        qd = to_dev(step_q(w, 0, len(live)), dtype)
        want = dense.decode(step_q(w, 0, len(live)), live)
        outs = [torch.full_like(qd, 3.0) for _ in range(3)]
        for chunk in (512, 16):  # whole units, and chunks that leave partial results for the merge
            ap.apar_set_chunk_blocks(h, chunk)
            ap.apar_decode_attention(h, qd, live, outs[0])
            ap.apar_decode_attention(h, qd, live, outs[1])
            ap.apar_decode_attention_fixed(h, qd, live, outs[2])
            torch.cuda.synchronize()
            assert_close(to_host(outs[0]), want, dtype, f"chunk {chunk}")
            assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
        if n_q == 5 or dtype == "bf16_fp8kv":
            return
        # candidates are folded in by one slice only
        c = 3
        q, ck, cv = spec_step_qkv(w, 1, len(live), c)
        rng = np.random.default_rng(1)
        masks = np.array([mask_rows_from_parents(draw_candidate_tree(rng, c)) for _ in live], dtype=np.uint8)
        for chunk in (512, 16):
            ap.apar_set_chunk_blocks(h, chunk)
            out = torch.empty_like(to_dev(q, dtype))
            ap.apar_decode_attention_spec(h, to_dev(q, dtype), to_dev(ck, dtype), to_dev(cv, dtype), torch.from_numpy(masks).cuda(), c, live, out)
            torch.cuda.synchronize()
            assert_close(to_host(out), dense.decode_spec(q, ck, cv, masks, live), dtype, f"candidates, chunk {chunk}")
