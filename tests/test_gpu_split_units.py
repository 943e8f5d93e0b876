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


@pytest.mark.parametrize("blocks", [400, 290, 114])
def test_short_rooms(blocks):
    """Row states have an eighth of the pool: seventy leaves below 640 rows on 16 kv heads leave too many for the smaller
    pools, whose units are cut into fewer slices or not at all."""
    import torch

    lens = [640] + [1] * 70
    w = manual_tree([-1] + [0] * 70, lens, HeadConfig(16, 16, 128, "bf16"), seed=5)
    dense = DenseThreads(16, 16, 128)
    with pool_for(w, blocks) as pool:
        pool.kv.fill_(0xFF)
        live, _ = replay_trace(w, pool, None, dense)
        q = step_q(w, 0, len(live))
        for call in (ap.apar_decode_attention, ap.apar_decode_attention_fixed, ap.apar_decode_attention):
            out = torch.full_like(to_dev(q, "bf16"), 3.0)
            call(pool.handle, to_dev(q, "bf16"), live, out)
            torch.cuda.synchronize()
            assert_close(to_host(out), dense.decode(q, live), "bf16", f"{call.__name__}, {blocks} blocks")


def test_fixed_entry_point_leaves_units_whole_where_the_tables_do_not_fit():
    """26 k one-row threads bring the tables to the fixed workspace's limit: the long thread beside them is cut by the other
    entry point only."""
    import torch

    n, long = 26000, 16000
    rng = np.random.default_rng(8)
    with ap.Pool(1, 1, 128, "bf16", n + long // 16 + 8, max_threads=n + 8) as pool:
        h = pool.handle
        live = [ap.apar_thread_create(h) for _ in range(n + 1)]
        k, v, k1, v1 = (to_dev(rng.standard_normal((m, 1, 128)).astype(np.float32), "bf16") for m in (long, long, n, n))
        ap.apar_append_kv(h, live[0], k, v)
        ap.apar_append_kv_batch(h, live[1:], k1, v1)
        q = to_dev(rng.standard_normal((n + 1, 1, 128)).astype(np.float32), "bf16")
        outs = [torch.full_like(q, 3.0) for _ in range(2)]
        ap.apar_decode_attention(h, q, live, outs[0])
        ap.apar_decode_attention_fixed(h, q, live, outs[1])
        torch.cuda.synchronize()
        want = torch.softmax(q[0].double() @ k[:, 0].double().T / 128 ** 0.5, dim=-1) @ v[:, 0].double()
        for out in outs:
            assert_close(to_host(out[:1]), want[None].cpu().numpy(), "bf16", "the long thread")
            assert torch.equal(out[1:], v1)  # (one row each: its value)


def test_partial_results_beyond_the_memory_side_cache():
    """More than 256 MiB of partial results (written with other stores than fewer): the merged rows are those of the same
    threads attended whole."""
    import torch

    n, length = 5500, 40
    with ap.Pool(32, 8, 128, "bf16", n * 3 + 8, max_threads=n + 8) as pool:
        h = pool.handle
        k, v = (torch.randn(length, n, 8, 128, device="cuda:0").bfloat16() for _ in "kv")
        live = [ap.apar_thread_create(h) for _ in range(n)]
        for i in range(length):
            ap.apar_append_kv_batch(h, live, k[i], v[i])
        q = torch.randn(n, 32, 128, device="cuda:0").bfloat16()
        outs = []
        for chunk in (1, 512):
            ap.apar_set_chunk_blocks(h, chunk)
            outs.append(torch.full_like(q, 3.0))
            ap.apar_decode_attention(h, q, live, outs[-1])
            rows = ap.apar_last_plan_info(h).n_partial_rows
            assert rows * 32 * 130 * 4 > 256 << 20 if chunk == 1 else rows == 0
        torch.cuda.synchronize()
        assert_close(to_host(outs[0]), to_host(outs[1]), "bf16")
