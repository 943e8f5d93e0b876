"""Calls of few units (on 16-bit pools they have a kernel of their own): list lengths around the tiles that kernel keeps on
their way, full, open and no tiles per wavefront, one to sixteen rows per unit, trees of two to four units, slices from two to
the most, against the dense oracle; the entry point that allocates nothing gives the same bits."""
import numpy as np
import pytest

import paper_2401_06761_amd as ap
from apar_workloads import HeadConfig, draw_candidate_tree, manual_tree, mask_rows_from_parents, spec_step_qkv, step_q
from oracle import DenseThreads

from harness import assert_close, blocks_upper_bound, pool_for, replay_trace, to_dev, to_host

pytestmark = pytest.mark.gpu

# q heads, kv heads, (prompt, leaves) of every tree
CALLS = {
    "one_block": (1, 1, [(1, [1])]),
    "tiles_1_to_9": (2, 2, [(16 * n + n % 3, [1]) for n in range(1, 10)]),
    "full_tiles_only": (2, 2, [(16 * n, [16]) for n in (15, 16, 17, 24, 31)]),
    "open_tiles_only": (2, 2, [(1, [1] * 15), (3, [2] * 13 + [15])]),
    "rows_1_15_16": (1, 1, [(300, [7]), (250, list(range(1, 16))), (280, list(range(10, 26)))]),
    "units_of_a_tree": (8, 2, [(200, [5, 16, 17, 31, 32]), (90, [40] * 9), (33, list(range(20, 36)))]),
    "group_16": (16, 1, [(150, [3, 16, 33, 20])]),
    "group_5": (5, 1, [(210, [1 + 9 * k for k in range(10)])]),
    "slices": (2, 2, [(2500, [1, 20, 33])]),
    "most_slices": (1, 1, [(11000, [40] * 17)]),
    "wide_trees": (32, 8, [(100, [9 * k + 1 for k in range(23)]), (47, [30] * 17)]),
    "more_than_compute_units": (16, 16, [(20 + k, [1 + k % 40] * 3) for k in range(60)]),
    "one_long_among_many": (16, 16, [(3000, [30] * 3)] + [(20 + k, [1 + k % 40] * 3) for k in range(40)]),
    "two_row_tiles": (64, 8, [(6000, [40] * 8), (33, [20] * 3), (500, [5, 90, 17, 16, 1])]),
    "two_row_tiles_in_slices": (64, 8, [(16 * 700, [40] * 7)]),
    "as_many_as_compute_units": (32, 32, [(60 + 9 * k, [4 + k] * 4) for k in range(8)]),
}


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16_fp8kv", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("call", list(CALLS))
def test_against_the_oracle(dtype, d, call):
    import torch

    n_q, n_kv, trees = CALLS[call]
    parents, lens = [], []
    for prompt, leaves in trees:
        root = len(parents)
        parents += [-1] + [root] * len(leaves)
        lens += [prompt] + leaves
    w = manual_tree(parents, lens, HeadConfig(n_q, n_kv, d, dtype), seed=9)
    dense = DenseThreads(n_q, n_kv, d)
    with pool_for(w, blocks_upper_bound(w)) as pool:
        pool.kv.fill_(0xFF)
        h = pool.handle
        live, _ = replay_trace(w, pool, None, dense)
        q = step_q(w, 0, len(live))
        outs = [torch.full_like(to_dev(q, dtype), 3.0) for _ in range(3)]
        ap.apar_decode_attention(h, to_dev(q, dtype), live, outs[0])
        ap.apar_decode_attention(h, to_dev(q, dtype), live, outs[1])
        ap.apar_decode_attention_fixed(h, to_dev(q, dtype), live, outs[2])
        torch.cuda.synchronize()
        wgs = np.asarray(ap.apar_last_plan_export(h, ap.APAR_PLAN_WORKGROUPS)).reshape(-1, 32)
        assert all(wg[1] == 0 for wg in wgs) and len(wgs) * n_kv <= 1024
        assert ({wg[3] & 255 for wg in wgs} == {1}) == (dtype == "f32" or call[:3] != "two" or (dtype == "bf16_fp8kv" and call == "two_row_tiles"))
        assert_close(to_host(outs[0]), dense.decode(q, live), dtype)
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
        c = 3
        if c * n_q // n_kv > 16 or dtype == "bf16_fp8kv":
            return
        q, ck, cv = spec_step_qkv(w, 1, len(live), c)
        rng = np.random.default_rng(1)
        masks = np.array([mask_rows_from_parents(draw_candidate_tree(rng, c)) for _ in live], dtype=np.uint8)
        out = torch.full_like(to_dev(q, dtype), 3.0)
        ap.apar_decode_attention_spec(h, to_dev(q, dtype), to_dev(ck, dtype), to_dev(cv, dtype), torch.from_numpy(masks).cuda(), c, live, out)
        torch.cuda.synchronize()
        assert_close(to_host(out), dense.decode_spec(q, ck, cv, masks, live), dtype, "candidates")


@pytest.mark.parametrize("dtype", ["bf16", "bf16_fp8kv", "f32"])
@pytest.mark.parametrize("n_q,n_kv,cand,n_trees,row_tiles", [(4, 2, 1, 3, 1), (4, 2, 4, 3, 1), (32, 2, 2, 3, 1), (40, 40, 4, 13, 2), (40, 40, 1, 25, 1)])
def test_trees_of_two_fork_levels(dtype, n_q, n_kv, cand, n_trees, row_tiles):
    """Segments below the top lie in one unit or across several; candidates on every pool type; 26 units of 16 rows x 40 heads are too many."""
    import torch

    parents, lens = [], []
    for k in range(n_trees):  # eight threads: three of the prompt's children, five of its fourth
        r = len(parents)
        parents += [-1, r, r, r, r] + [r + 4] * 5
        lens += [33 + 7 * k, 16, 5, 40, 50 + k, 1, 17, 30, 16, 9]
    w = manual_tree(parents, lens, HeadConfig(n_q, n_kv, 128, dtype), seed=6)
    dense = DenseThreads(n_q, n_kv, 128)
    with pool_for(w, blocks_upper_bound(w)) as pool:
        pool.kv.fill_(0xFF)
        h = pool.handle
        live, _ = replay_trace(w, pool, None, dense)
        assert len(live) == 8 * n_trees
        q, ck, cv = spec_step_qkv(w, 1, len(live), cand)
        rng = np.random.default_rng(1)
        masks = np.array([mask_rows_from_parents(draw_candidate_tree(rng, cand)) for _ in live], dtype=np.uint8)
        outs = [torch.full_like(to_dev(q, dtype), 3.0) for _ in range(2)]
        for out in outs:
            ap.apar_decode_attention_spec(h, to_dev(q, dtype), to_dev(ck, dtype), to_dev(cv, dtype), torch.from_numpy(masks).cuda(), cand, live, out)
        torch.cuda.synchronize()
        wgs = np.asarray(ap.apar_last_plan_export(h, ap.APAR_PLAN_WORKGROUPS)).reshape(-1, 32)
        if row_tiles == 1 or dtype != "f32":  # (fp32 pools have no wider units)
            assert all(wg[1] == 0 for wg in wgs) and {wg[3] & 255 for wg in wgs} == {row_tiles}
        assert_close(to_host(outs[0]), dense.decode_spec(q, ck, cv, masks, live), dtype, "candidates")
        assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("dtype", ["bf16", "bf16_fp8kv", "f32"])
@pytest.mark.parametrize("n_q,n_kv,trees,shared", [
    (32, 4, [(33600, [40] * 6), (100, [30] * 3)], True),              # a long tree of 48 rows: the general plan for every tree
    (8, 4, [(33600, [40, 3]), (100, [30] * 11), (16, [1])], False),   # of 4 rows: chunks without a shared list, merged
])
def test_trees_that_stand_alone_for_their_blocks(dtype, n_q, n_kv, trees, shared):
    import torch

    parents, lens = [], []
    for prompt, leaves in trees:
        root = len(parents)
        parents += [-1] + [root] * len(leaves)
        lens += [prompt] + leaves
    w = manual_tree(parents, lens, HeadConfig(n_q, n_kv, 128, dtype), seed=4)
    dense = DenseThreads(n_q, n_kv, 128)
    with pool_for(w, blocks_upper_bound(w)) as pool:
        pool.kv.fill_(0xFF)
        h = pool.handle
        live, _ = replay_trace(w, pool, None, dense)
        q, ck, cv = spec_step_qkv(w, 1, len(live), 2)
        masks = np.array([[1, 3]] * len(live), dtype=np.uint8)
        out = torch.full_like(to_dev(q, dtype), 3.0)
        ap.apar_decode_attention_spec(h, to_dev(q, dtype), to_dev(ck, dtype), to_dev(cv, dtype), torch.from_numpy(masks).cuda(), 2, live, out)
        wgs = np.asarray(ap.apar_last_plan_export(h, ap.APAR_PLAN_WORKGROUPS)).reshape(-1, 32)
        assert ap.apar_last_plan_info(h).n_partial_rows > 0 and any(wg[1] > 0 for wg in wgs) == shared
        assert_close(to_host(out), dense.decode_spec(q, ck, cv, masks, live), dtype, "candidates")
        q = step_q(w, 0, len(live))
        outs = [torch.full_like(to_dev(q, dtype), 3.0) for _ in range(2)]
        ap.apar_decode_attention(h, to_dev(q, dtype), live, outs[0])
        ap.apar_decode_attention_fixed(h, to_dev(q, dtype), live, outs[1])
        torch.cuda.synchronize()
        wgs = np.asarray(ap.apar_last_plan_export(h, ap.APAR_PLAN_WORKGROUPS)).reshape(-1, 32)
        assert ap.apar_last_plan_info(h).n_partial_rows > 0 and any(wg[1] > 0 for wg in wgs) == shared
        assert_close(to_host(outs[0]), dense.decode(q, live), dtype)
        assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("prompt", [500, 2500, 4100, 11000])  # 2 to 43 slices
def test_an_infinity_in_every_slice_stays_one(dtype, prompt):
    """Zero queries weigh every row alike: a dim that holds an infinity in each full block of the prompt comes out infinite, the others
    as the mean of their values, however many slices the unit is folded from."""
    import torch

    n_kv, d = 2, 128
    with ap.Pool(n_kv, n_kv, d, dtype, 1024, max_threads=16) as pool:
        h = pool.handle
        rng = np.random.default_rng(prompt)
        k, v = rng.standard_normal((2, prompt, n_kv, d))
        v[3::16, :, 5] = np.inf
        v[prompt // 16 * 16:, :, 5] = 1.0
        root = ap.apar_thread_create(h)
        ap.apar_append_kv(h, root, to_dev(k, dtype), to_dev(v, dtype), prompt)
        live = [root] + ap.apar_fork(h, root, 2)
        out = to_dev(np.zeros((3, n_kv, d)), dtype)
        ap.apar_decode_attention(h, to_dev(np.zeros((3, n_kv, d)), dtype), live, out)
        got = to_host(out)
        assert (got[:, :, 5] == np.inf).all()
        want = to_host(to_dev(v, dtype)).astype(np.float64).mean(0)
        rest = np.arange(d) != 5
        assert_close(got[:, :, rest], np.broadcast_to(want[:, rest], (3, n_kv, d - 1)), dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n_q,n_kv,cand", [(16, 2, 3), (8, 1, 8), (64, 8, 4), (10, 2, 5), (640, 40, 4)])
def test_threads_of_more_rows_than_a_unit_holds(dtype, n_q, n_kv, cand):
    import torch

    leaves = [1, 16, 17, 40, 90]
    w = manual_tree([-1] + [0] * 5 + [-1, 6, 6], [170] + leaves + [16, 3, 50], HeadConfig(n_q, n_kv, 128, dtype), seed=2)
    dense = DenseThreads(n_q, n_kv, 128)
    with pool_for(w, blocks_upper_bound(w)) as pool:
        pool.kv.fill_(0xFF)
        h = pool.handle
        live, _ = replay_trace(w, pool, None, dense)
        q, ck, cv = spec_step_qkv(w, 1, len(live), cand)
        rng = np.random.default_rng(1)
        masks = np.array([mask_rows_from_parents(draw_candidate_tree(rng, cand)) for _ in live], dtype=np.uint8)
        outs = [torch.full_like(to_dev(q, dtype), 3.0) for _ in range(2)]
        for out in outs:
            ap.apar_decode_attention_spec(h, to_dev(q, dtype), to_dev(ck, dtype), to_dev(cv, dtype), torch.from_numpy(masks).cuda(), cand, live, out)
        torch.cuda.synchronize()
        wgs = np.asarray(ap.apar_last_plan_export(h, ap.APAR_PLAN_WORKGROUPS)).reshape(-1, 32)
        slices = -(-cand * n_q // n_kv // 16)
        if n_kv < 40 or dtype != "f32":  # (1280 units of 16 rows are too many, and fp32 pools have no wider ones)
            assert all(wg[1] == 0 for wg in wgs) and sum(wg[7] for wg in wgs) == len(live) * slices
            assert {wg[3] & 255 for wg in wgs} == {2 if n_kv == 40 else 1}
        assert_close(to_host(outs[0]), dense.decode_spec(q, ck, cv, masks, live), dtype)
        assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("dtype", ["bf16", "bf16_fp8kv", "f32"])
@pytest.mark.parametrize("n_q,n_kv,cand,root", [(16, 2, 4, 40), (16, 2, 3, 900)])  # (tables with the arguments, and staged ones)
def test_a_loop_carries_threads_of_more_rows_than_a_unit(dtype, n_q, n_kv, cand, root):
    import torch

    w = manual_tree([-1] + [0] * 3, [root, 1, 15, 40], HeadConfig(n_q, n_kv, 128, dtype), seed=2)
    dense = DenseThreads(n_q, n_kv, 128)
    with pool_for(w, blocks_upper_bound(w) + 32) as pool:
        h = pool.handle
        live, _ = replay_trace(w, pool, None, dense)
        for step in range(20):
            q, ck, cv = spec_step_qkv(w, step, len(live), cand)
            masks = np.array([[1, 3, 5, 9][:cand]] * len(live), dtype=np.uint8)
            out = torch.full_like(to_dev(q, dtype), 3.0)
            ap.apar_decode_attention_spec(h, to_dev(q, dtype), to_dev(ck, dtype), to_dev(cv, dtype), torch.from_numpy(masks).cuda(), cand, live, out)
            torch.cuda.synchronize()
            assert_close(to_host(out), dense.decode_spec(q, ck, cv, masks, live), dtype, f"step {step}")
            accept = np.full(len(live), 1, dtype=np.uint8)
            ap.apar_commit_candidates(h, live, to_dev(ck, dtype), to_dev(cv, dtype), cand, accept)
            dense.commit_candidates(live, ck, cv, accept)
        assert all(wg[1] == 0 for wg in np.asarray(ap.apar_last_plan_export(h, ap.APAR_PLAN_WORKGROUPS)).reshape(-1, 32))
        assert ap.apar_plan_counts(h) == (1, 19)


@pytest.mark.parametrize("dtype", ["bf16", "bf16_fp8kv"])
@pytest.mark.parametrize("n_kv,group,trees", [(1, 1, [(60, [5, 16, 17])]), (2, 4, [(1500, [20, 3])]), (40, 4, [(40, [9, 1, 16, 17, 8])] * 13),
                                              (1, 1, [(300, [5] * 20)] * 3)])
def test_packed_tables_give_the_same_bits(dtype, n_kv, group, trees):
    """Tables that go along packed, as they are (pools of more than 2^18 blocks) and staged: one and two row tiles, slices, packed ones that
    would not fit otherwise."""
    import torch

    outs = []
    for blocks in (4096, (1 << 18) + 1):
        if blocks * n_kv > 1 << 20:
            continue  # (80 GiB)
        with ap.Pool(n_kv * group, n_kv, 128, dtype, blocks, max_threads=4096) as pool:
            h = pool.handle
            gen = torch.Generator(device="cuda")
            gen.manual_seed(3)
            rand = lambda n, heads=n_kv: torch.randn((n, heads, 128), generator=gen, device="cuda").to(torch.bfloat16)
            live = []
            for prompt, leaves in trees:
                root = ap.apar_thread_create(h)
                ap.apar_append_kv(h, root, rand(prompt), rand(prompt))
                kids = ap.apar_fork(h, root, len(leaves))
                for t, n in zip(kids, leaves):
                    ap.apar_append_kv(h, t, rand(n), rand(n))
                live += kids
            q = rand(len(live), n_kv * group)
            for call in (ap.apar_decode_attention, ap.apar_decode_attention_fixed):
                outs.append(torch.full_like(q, 3.0))
                call(h, q, live, outs[-1])
            torch.cuda.synchronize()
            assert all(wg[1] == 0 for wg in np.asarray(ap.apar_last_plan_export(h, ap.APAR_PLAN_WORKGROUPS)).reshape(-1, 32))
    assert not (outs[0] == 3.0).any() and all(torch.equal(outs[0], o) for o in outs)
