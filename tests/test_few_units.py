"""Plans of calls with few units: trees of up to four units of 16 rows are cut by rank into units without shared
lists, whose tiles are level over the four wavefronts; wider trees, many trees and trees that would be read too often go the
general way, as every tree does with the knob that cuts by rank switched off.  Every plan shows every row its blocks, and a
decode loop carries it over."""
import numpy as np
import pytest

import paper_2401_06761_amd as ap

from harness import PlanTablesOnDevice, check_plan_covers_tables


def grow(h, prompt, leaves, root=None):
    """A tree's threads; a leaf that is itself (tokens, leaves) forks again."""
    if root is None:
        root = ap.apar_thread_create(h)
    ap.apar_append_kv(h, root, None, None, prompt)
    kids, live = ap.apar_fork(h, root, len(leaves)), []
    ap.apar_free_thread(h, root)
    for t, leaf in zip(kids, leaves):
        if isinstance(leaf, tuple):
            live += grow(h, *leaf, root=t)
        else:
            ap.apar_append_kv(h, t, None, None, leaf)
            live.append(t)
    return live


def workgroups(h):
    return np.asarray(ap.apar_last_plan_export(h, ap.APAR_PLAN_WORKGROUPS)).reshape(-1, 32)


def every_row_group_once(h, live, slices):
    """Every slice of every thread is in one direct unit, which lists each block of the thread's table once."""
    wgs = workgroups(h)
    tiles = np.asarray(ap.apar_last_plan_export(h, ap.APAR_PLAN_TILES)).reshape(-1, 2)
    dfs = ap.apar_last_plan_export(h, ap.APAR_PLAN_DFS_THREADS)
    assert sorted(g for wg in wgs for g in range(wg[6], wg[6] + wg[7])) == list(range(len(live) * slices))
    assert ap.apar_last_plan_info(h).n_partial_rows == 0
    for wg in wgs:
        assert wg[6] // slices == (wg[6] + wg[7] - 1) // slices and wg[3] & 255 == wg[7]  # (a row tile per slice, of one thread)
        thread = live[dfs[wg[6] // slices]]
        table, length, got = ap.apar_thread_block_table(h, thread), ap.apar_thread_len(h, thread), []
        for k in range(4):
            ofs, n, lo, groups, _, flags = wg[4 + 6 * k:10 + 6 * k]
            assert lo == wg[6] and groups == wg[7] and flags == 3
            fills = [int(m) >> 20 & 31 for _, m in tiles[ofs:ofs + n]]
            assert all(int(m) & 0xfffff == groups << 10 for _, m in tiles[ofs:ofs + n]) and [f == 16 for f in fills] == [i < wg[28 + k] for i in range(n)]
            got += [(int(b), f) for (b, _), f in zip(tiles[ofs:ofs + n], fills)]
        # (a block that is not the last is full)
        assert sorted(got) == sorted((b, min(16, length - 16 * i)) for i, b in enumerate(table))


# kv heads, q heads per kv head, (prompt, leaves) per tree, row tiles of the units by data type (0: not a call of few units)
BF16, FP8, F32 = "bf16", "bf16_fp8kv", "f32"
CALLS = [
    (2, 1, [(300, [20 + k for k in range(17)])], {BF16: 1, FP8: 1, F32: 1}),           # 17 rows: two units
    (2, 1, [(300, [5] * 64)], {BF16: 1, FP8: 1, F32: 1}),
    (2, 1, [(300, [5] * 65)], {BF16: 0, FP8: 0, F32: 0}),                                # five units of sixteen threads
    (8, 4, [(100, [30] * 5), (17, [1, 16, 17, 40, 8, 90])], {BF16: 1, FP8: 1, F32: 1}),
    (8, 16, [(64, [9, 16, 33])], {BF16: 1, FP8: 1, F32: 1}),
    (8, 5, [(64, [9, 16, 33, 1, 70])], {BF16: 1, FP8: 1, F32: 1}),
    (8, 1, [(40, [10] * 20)] * 64, {BF16: 1, FP8: 1, F32: 1}),                           # 128 units x 8 heads
    (8, 1, [(40, [10] * 20)] * 65, {BF16: 2, FP8: 2, F32: 0}),                           # (130; 65 of two row tiles)
    (8, 1, [(40, [10] * 20)] * 129, {BF16: 0, FP8: 0, F32: 0}),
    (8, 4, [(40, [10] * 30)] * 2, {BF16: 1, FP8: 1, F32: 1}),                            # eight units each, of four threads
    (8, 8, [(16 * 590, [40] * 8)], {BF16: 2, FP8: 1, F32: 1}),                           # three more readers of 590 tiles x 64 KiB
    (8, 8, [(16 * 1000, [40] * 8)], {BF16: 2, FP8: 2, F32: 1}),
    (8, 8, [(16 * 1000, [40] * 16)], {BF16: 0, FP8: 2, F32: 1}),                         # (and three of two row tiles)
    (8, 8, [(16 * 1008, [40] * 8)], {BF16: 0, FP8: 2, F32: 1}),                          # 64 rows: 63 MiB again of 64.5 (1008 tiles of 1032)
    (8, 8, [(16 * 1008, [40] * 9)], {BF16: 0, FP8: 2, F32: 1}),                          # 72 rows: 126 MiB
    (8, 8, [(16 * 880, [40] * 9)], {BF16: 2, FP8: 2, F32: 1}),                           # 110
    (8, 8, [(2048, [40] * 8)] * 8, {BF16: 0, FP8: 2, F32: 1}),
    (1, 8, [(16 * 130, [20] * 32)], {BF16: 0, FP8: 1, F32: 1}),                          # 256 rows below 130 blocks: the matrix kernel's
    (1, 1, [(16 * 2100, [1] * 18)], {BF16: 0, FP8: 0, F32: 0}),                          # more tiles than a unit may list
]


@pytest.mark.parametrize("dtype", [BF16, FP8, F32])
@pytest.mark.parametrize("n_kv,group,trees,few", CALLS)
def test_plans_of_few_units(dtype, n_kv, group, trees, few):
    blocks = sum(p // 16 + 2 + sum(n // 16 + 2 for n in leaves) for p, leaves in trees)
    with ap.Pool(n_kv * group, n_kv, 128, dtype, blocks, max_threads=4096, dry_run=True) as pool:
        h = pool.handle
        live = [t for prompt, leaves in trees for t in grow(h, prompt, leaves)]
        ap.apar_decode_attention(h, None, live, None)
        check_plan_covers_tables(h, live, n_kv, group)
        wgs = workgroups(h)
        per_unit = max(1, few[dtype]) * (16 // group)
        units = sum(-(-len(leaves) // per_unit) for _, leaves in trees)
        shared = any(wg[1] > 0 for wg in wgs)
        if few[dtype]:
            assert not shared and len(wgs) == units and max(wg[3] & 255 for wg in wgs) == few[dtype]
            for wg in wgs:
                tiles, full = [wg[5 + 6 * k] for k in range(4)], wg[28:32]
                assert all(wg[9 + 6 * k] & 2 for k in range(4)) and max(tiles) - min(tiles) <= 1 + max(t - f for t, f in zip(tiles, full))
        else:
            assert shared or ap.apar_last_plan_info(h).n_partial_rows > 0
        ap.apar_set_inline_shared(h, False)  # nothing is cut by rank
        ap.apar_decode_attention(h, None, live, None)
        check_plan_covers_tables(h, live, n_kv, group)


# Trees of more blocks than a unit may list (2048), whose top segment stands alone: kv heads, q heads per kv head, candidates, trees, and whether
# the call still is one of few units (trees of one row tile: chunks without a shared list)
LONG = [
    (8, 8, 1, [(33600, [40] * 3), (100, [30] * 3)], False),
    (4, 8, 1, [(33600, [40] * 6), (100, [30] * 3)], False),
    (8, 4, 1, [(33000, [40] * 6), (100, [30] * 6)], False),
    (8, 4, 1, [(33000, [40] * 5), (500, [30] * 8)], False),
    (8, 4, 1, [(60000, [40] * 5), (500, [30] * 8)], False),
    (8, 4, 1, [(40000, [50, (90, [20] * 6), 70])], False),
    (1, 4, 1, [(40000, [(60, [20] * 6), (75, [30] * 6)])], False),
    (8, 1, 1, [(40000, [(60, [20] * 20), (75, [30] * 20)])], False),
    (8, 5, 1, [(33000, [20] * 4), (40, [16] * 7)], False),
    (1, 1, 1, [(16 * 2100, [1] * 18), (300, [5] * 20)], False),
    (8, 8, 3, [(33000, [40] * 2), (100, [30])], False),            # two slices per thread
    (8, 4, 1, [(33600, [40] * 2), (100, [30] * 3)], True),
    (8, 4, 1, [(33600, [40] * 2), (100, [30] * 6), (16 * 300, [9] * 4)], True),
    (1, 1, 1, [(40000, [50, (70000, [20] * 6), 70])], True),
]


@pytest.mark.parametrize("dtype", [BF16, FP8, F32])
@pytest.mark.parametrize("n_kv,group,cand,trees,few", LONG)
def test_trees_that_stand_alone_for_their_blocks(dtype, n_kv, group, cand, trees, few):
    with ap.Pool(n_kv * group, n_kv, 128, dtype, 16384, max_threads=256, dry_run=True) as pool:
        h = pool.handle
        attend = lambda: ap.apar_decode_attention_spec(h, None, None, None, None, cand, live, None)
        live = [t for prompt, leaves in trees for t in grow(h, prompt, leaves)]
        attend()
        check_plan_covers_tables(h, live, n_kv, cand * group)
        tables = range(ap.APAR_PLAN_WORKGROUPS, ap.APAR_PLAN_GEOMETRY + 1)
        plan = [list(ap.apar_last_plan_export(h, k)) for k in tables]
        assert ap.apar_last_plan_info(h).n_partial_rows > 0
        if few:
            assert all(wg[1] == 0 and wg[3] & 255 <= 2 for wg in workgroups(h))
            ap.apar_append_kv_batch(h, live, None, None)
            attend()
            check_plan_covers_tables(h, live, n_kv, cand * group)
        else:  # the plan of a pool that makes none of few units
            ap.apar_set_inline_shared(h, True)
            attend()
            assert ap.apar_plan_counts(h)[0] == 2 and plan == [list(ap.apar_last_plan_export(h, k)) for k in tables]


@pytest.mark.parametrize("dtype", [BF16, FP8, F32])
def test_a_pool_whose_knobs_were_set_plans_by_them(dtype):
    """The knob of the matrix kernel counts on the pools that have that kernel: others ignore it."""
    with ap.Pool(8, 2, 128, dtype, 256, max_threads=64, dry_run=True) as pool:
        h = pool.handle
        live = grow(h, 300, [30] * 6)

        def few():
            ap.apar_decode_attention(h, None, live, None)
            check_plan_covers_tables(h, live, 2, 4)
            return all(wg[1] == 0 and wg[3] & 255 == 1 for wg in workgroups(h))

        assert few()
        ap.apar_set_matrix_units(h, 1, 1)
        assert few() == (dtype != BF16)
        ap.apar_set_chunk_blocks(h, 512)
        assert not few()


@pytest.mark.parametrize("dtype", [BF16, FP8, F32])
@pytest.mark.parametrize("n_kv,group,cand,n_trees,tree", [
    # a leaf beside a long paragraph that forks four times: cut by rank into 2 + 3 threads, the paragraph lies in both units
    (8, 4, 1, 1, (32, [16, (16000, [9, 8, 7, 6])])),
    (8, 4, 1, 8, (32, [16, (16000, [9, 8, 7, 6])])),
    (8, 4, 1, 60, (32, [16, (16000, [9, 8, 7, 6])])),
    (1, 4, 1, 60, (32, [16, (16000, [9, 8, 7, 6])])),
    (8, 8, 1, 8, (160, [(4000, [9, 8]), 16, (8000, [9, 8])])),
    (2, 1, 1, 40, (48, [(900, [5] * 15), (1700, [6] * 9), (33, [7] * 13)])),
    (8, 8, 5, 10, (640, [(900, [5] * 3), 4])),
])
def test_tiles_that_several_units_list(dtype, n_kv, group, cand, n_trees, tree):
    """What units of few may list and list again is what they do list, whichever units a segment of the trees lies in."""
    with ap.Pool(n_kv * group, n_kv, 128, dtype, 1 << 17, max_threads=4096, dry_run=True) as pool:
        h = pool.handle
        live = [t for _ in range(n_trees) for t in grow(h, *tree)]
        ap.apar_decode_attention_spec(h, None, None, None, None, cand, live, None)
        wgs, info = workgroups(h), ap.apar_last_plan_info(h)
        if any(wg[1] > 0 for wg in wgs) or info.n_partial_rows > 0:
            return
        assert dtype == F32 or len(wgs) * n_kv <= 1024
        listed = sum(wg[5 + 6 * k] for wg in wgs for k in range(4))
        assert listed <= 65536
        # on 16-bit pools 56 MiB, 112 where there are units of two row tiles
        limit = {BF16: 56 << 20, FP8: 112 << 20, F32: 1 << 60}[dtype] // (n_kv * 8192) << int(max(wg[3] & 255 for wg in wgs) - 1)
        assert listed - info.unique_blocks <= limit


@pytest.mark.parametrize("seed", range(6))
def test_a_loop_carries_them(seed):
    rng = np.random.default_rng(seed)
    n_kv, group = int(rng.choice([1, 2, 8])), int(rng.choice([1, 2, 4, 8]))
    with ap.Pool(n_kv * group, n_kv, 128, "bf16", 4096, max_threads=1 << 20, dry_run=True) as pool:
        h = pool.handle
        live = []
        for _ in range(int(rng.integers(1, 5))):
            live += grow(h, int(rng.integers(1, 400)), [int(x) for x in rng.integers(1, 60, size=int(rng.integers(16 // group + 1, 64 // group + 1)))])
        for step in range(60):
            if step:
                ap.apar_append_kv_batch(h, live, None, None)
                pos = int(rng.integers(0, len(live)))
                (child,) = ap.apar_fork(h, live[pos], 1)  # a thread finishes and one forked from it carries on in its place
                ap.apar_free_thread(h, live[pos])
                live[pos] = child
            ap.apar_decode_attention(h, None, live, None)
            check_plan_covers_tables(h, live, n_kv, group)
            assert all(wg[1] == 0 and wg[3] & 255 == 1 for wg in workgroups(h))
        built, carried = ap.apar_plan_counts(h)
        assert built + carried == 60 and built <= 2


@pytest.mark.parametrize("n_kv,group,cand,few", [(8, 8, 3, 1), (1, 8, 8, 1), (8, 16, 4, 1), (2, 5, 5, 1), (16, 16, 4, 2), (16, 8, 5, 1), (32, 16, 4, 0)])
def test_threads_of_more_rows_than_a_unit_holds(n_kv, group, cand, few):
    """A unit per slice of every thread, or per two; a call with the same list carries the plan over."""
    with ap.Pool(n_kv * group, n_kv, 128, "bf16", 2048, max_threads=256, dry_run=True) as pool:
        h = pool.handle
        live = grow(h, 70, [1, 16, 17, 40, 90]) + grow(h, 16, [3, 50]) + grow(h, 5, [20] * 12)
        spec = lambda: ap.apar_decode_attention_spec(h, None, None, None, None, cand, live, None)
        for step in range(3):
            spec()
            slices = -(-cand * group // 16)
            if few:
                every_row_group_once(h, live, slices)
            else:
                check_plan_covers_tables(h, live, n_kv, cand * group)
            assert (max(wg[3] & 255 for wg in workgroups(h)) if not any(wg[1] for wg in workgroups(h)) else 0) == few
            built = ap.apar_plan_counts(h)[0]
            spec()
            assert ap.apar_plan_counts(h)[0] == built
            ap.apar_append_kv_batch(h, live, None, None)


@pytest.mark.parametrize("n_kv,group,cand,row_tiles", [(8, 8, 4, 1), (1, 8, 8, 1), (2, 5, 5, 1), (16, 16, 4, 2), (16, 16, 3, 2)])
def test_a_loop_carries_threads_of_more_rows_than_a_unit(n_kv, group, cand, row_tiles):
    """Every one of a thread's units follows its last blocks: rows appended, blocks that fill up, copies on write."""
    with ap.Pool(n_kv * group, n_kv, 128, "bf16", 4096, max_threads=4096, dry_run=True) as pool:
        h = pool.handle
        live = grow(h, 70, [1, 16, 17, 40, 90, 31]) + (grow(h, 16, [3] * 18) if row_tiles == 2 else [])
        rng, on_device = np.random.default_rng(cand), PlanTablesOnDevice(h)
        for step in range(40):
            if step:
                ap.apar_append_kv_batch(h, live, None, None)
                pos = int(rng.integers(0, len(live)))
                (child,) = ap.apar_fork(h, live[pos], 1)
                ap.apar_free_thread(h, live[pos])
                live[pos] = child
            ap.apar_decode_attention_spec(h, None, None, None, None, cand, live, None)
            every_row_group_once(h, live, -(-cand * group // 16))
            on_device.follow()
            assert max(wg[3] & 255 for wg in workgroups(h)) == row_tiles
            info, blocks = ap.apar_last_plan_info(h), {}
            for t in live:
                n = ap.apar_thread_len(h, t)
                blocks.update({b: min(16, n - 16 * i) for i, b in enumerate(ap.apar_thread_block_table(h, t))})
            assert info.unique_blocks == len(blocks) and info.unique_tokens == sum(blocks.values())
            assert info.path_tokens == sum(ap.apar_thread_len(h, t) for t in live)
        built, carried = ap.apar_plan_counts(h)
        assert (built, carried) == (1, 39)
