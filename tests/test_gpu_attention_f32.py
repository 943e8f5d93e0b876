"""The fp32 attention kernel where its 16x16 tiles can go wrong: ranges of rows, slices, two row tiles per
wavefront, split units, causal tiles, candidates - and rows next to which another thread holds infinities or NaN."""
import numpy as np
import pytest

import paper_2401_06761_amd as ap
from apar_workloads import HeadConfig, manual_tree, step_q
from oracle import DenseThreads

from harness import assert_close, blocks_upper_bound, check_plan_covers_tables, pool_for, replay_trace, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_q,n_kv,fan", [(1, 1, 1), (2, 2, 15), (2, 2, 17), (4, 4, 65), (2, 2, 129), (16, 1, 3), (10, 2, 7), (6, 2, 40)])
def test_row_ranges_and_row_tiles(d, n_q, n_kv, fan):
    import torch

    parents, lens = [-1], [37]
    for i in range(fan):
        parents.append(0)
        lens.append(1 + (i * 11) % 50)
        if i % 3 == 1:
            parents += [len(parents) - 1] * 2
            lens += [16, 300 if i == 1 else 7]
    w = manual_tree(parents, lens, HeadConfig(n_q, n_kv, d, "f32"), seed=fan)
    dense = DenseThreads(n_q, n_kv, d)
    with pool_for(w, blocks_upper_bound(w)) as pool:
        pool.kv.fill_(0xFF)
        live, _ = replay_trace(w, pool, None, dense)
        q = step_q(w, 0, len(live))
        out = torch.empty_like(to_dev(q, "f32"))
        for chunk in (512, 3):  # whole units, and partial results
            ap.apar_set_chunk_blocks(pool.handle, chunk)
            ap.apar_decode_attention(pool.handle, to_dev(q, "f32"), live, out)
            torch.cuda.synchronize()
            check_plan_covers_tables(pool.handle, live, n_kv, n_q // n_kv)
            assert_close(to_host(out), dense.decode(q, live), "f32", f"chunk {chunk}")


@pytest.mark.parametrize("d,fan", [(64, 5), (128, 5), (128, 70)])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_a_threads_infinities_stay_its_own(d, fan, bad):
    """One leaf's rows hold infinities or NaN, in K or in V: its siblings' outputs are what they are without it."""
    import torch

    heads = HeadConfig(2, 2, d, "f32")
    w = manual_tree([-1] + [0] * fan, [40] + [9 + 3 * (i % 5) for i in range(fan)], heads, seed=1)
    for where in ("k", "v"):
        dense = DenseThreads(2, 2, d)
        with pool_for(w, blocks_upper_bound(w)) as pool:
            pool.kv.fill_(0xFF)
            live, _ = replay_trace(w, pool, None, dense)
            rng = np.random.default_rng(2)
            k, v = (rng.standard_normal((len(live), 2, d)).astype(np.float32) for _ in "kv")
            dense_k, dense_v = k.copy(), v.copy()
            (k if where == "k" else v)[2, :, 5] = bad
            ap.apar_append_kv_batch(pool.handle, live, to_dev(k, "f32"), to_dev(v, "f32"))
            for i, t in enumerate(live):
                dense.append(t, dense_k[i:i + 1], dense_v[i:i + 1])
            q = step_q(w, 0, len(live))
            out = torch.empty_like(to_dev(q, "f32"))
            ap.apar_decode_attention(pool.handle, to_dev(q, "f32"), live, out)
            # the same rows as the last two query tokens of a prefill call, whose first one must not see the last row
            m = [2] * len(live)
            q2 = np.repeat(q, 2, axis=0)
            out2 = torch.empty_like(to_dev(q2, "f32"))
            ap.apar_prefill_attention(pool.handle, to_dev(q2, "f32"), live, m, out2)
            torch.cuda.synchronize()
            got, want = to_host(out), dense.decode(q, live)
            got2, want2 = to_host(out2), dense.prefill(q2, live, m)
            others = [i for i in range(len(live)) if i != 2]
            assert_close(got[others], want[others], "f32", where)
            if where == "v" or np.isnan(bad):  # (an infinite key gives a logit of either infinity: a NaN, or a weight of 0)
                assert not np.isfinite(got[2]).all()
            rows = [r for r in range(2 * len(live)) if r != 5]
            assert_close(got2[rows], want2[rows], "f32", where)


@pytest.mark.parametrize("d", [64, 128])
def test_rows_at_any_four_byte_address(d):
    """fp32 rows are loaded and stored 16 bytes at a time; callers may hand over any float's address."""
    import torch

    w = manual_tree([-1, 0, 0], [21, 9, 30], HeadConfig(2, 2, d, "f32"), seed=4)
    dense = DenseThreads(2, 2, d)
    with pool_for(w, blocks_upper_bound(w)) as pool:
        pool.kv.fill_(0xFF)
        live, _ = replay_trace(w, pool, None, dense)
        rng = np.random.default_rng(3)
        k, v = (rng.standard_normal((len(live), 2, d)).astype(np.float32) for _ in "kv")

        def shifted(x):
            flat = torch.zeros(x.size + 1, dtype=torch.float32, device="cuda:0")
            flat[1:] = torch.from_numpy(x.reshape(-1)).cuda()
            return flat[1:].view(x.shape)

        ap.apar_append_kv_batch(pool.handle, live, shifted(k), shifted(v))
        for i, t in enumerate(live):
            dense.append(t, k[i:i + 1], v[i:i + 1])
        q = step_q(w, 0, len(live))
        out = shifted(np.zeros_like(q))
        ap.apar_decode_attention(pool.handle, shifted(q), live, out)
        torch.cuda.synchronize()
        assert_close(to_host(out), dense.decode(q, live), "f32")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("root", [40, 2100])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_logits_of_minus_infinity_beside_a_threads_infinities(d, root, bad):
    """Every sixteenth cached row, from the first on, has a logit of -inf for every query (weight 0), and one thread's V
    holds infinities or NaN: its siblings are what they are without it, on a short walk and on one that is cut into slices."""
    import torch

    n_leaf, hkv = 4, 2
    heads = HeadConfig(hkv, hkv, d, "f32")
    rng = np.random.default_rng(root + d)
    k, v = (rng.standard_normal((root, hkv, d)).astype(np.float32) for _ in "kv")
    k[::16, :, 7] = -np.inf
    dense = DenseThreads(hkv, hkv, d)
    w = manual_tree([-1], [1], heads, seed=1)
    with pool_for(w, 2 * (root // 16) + 16) as pool:
        pool.kv.fill_(0xFF)
        t = ap.apar_thread_create(pool.handle)
        assert t == dense.create()
        ap.apar_append_kv(pool.handle, t, to_dev(k, "f32"), to_dev(v, "f32"), root)
        dense.append(t, k, v)
        live = ap.apar_fork(pool.handle, t, n_leaf)
        assert list(live) == list(dense.fork(t, n_leaf))
        k1, v1 = (rng.standard_normal((n_leaf, hkv, d)).astype(np.float32) for _ in "kv")
        v1[2, :, 5] = bad
        ap.apar_append_kv_batch(pool.handle, live, to_dev(k1, "f32"), to_dev(v1, "f32"))
        for i, x in enumerate(live):
            dense.append(x, k1[i:i + 1], v1[i:i + 1])
        # and one whose own rows make slices of their own, an infinity or NaN among them
        k2, v2 = (rng.standard_normal((root, hkv, d)).astype(np.float32) for _ in "kv")
        k2[root // 3, :, 9] = bad
        v2[root // 2, :, 9] = bad
        ap.apar_append_kv(pool.handle, live[3], to_dev(k2, "f32"), to_dev(v2, "f32"), root)
        dense.append(live[3], k2, v2)
        q = rng.standard_normal((n_leaf, hkv, d)).astype(np.float32)
        q[:, :, 7] = 1.0 + np.abs(q[:, :, 7])
        want = dense.decode(q, live)
        others = [0, 1]
        for call in (ap.apar_decode_attention, ap.apar_decode_attention_fixed):
            out = torch.empty_like(to_dev(q, "f32"))
            call(pool.handle, to_dev(q, "f32"), live, out)
            torch.cuda.synchronize()
            got = to_host(out)
            assert_close(got[others], want[others], "f32", call.__name__)
            assert not np.isfinite(got[2]).all() and not np.isfinite(got[3]).all()
