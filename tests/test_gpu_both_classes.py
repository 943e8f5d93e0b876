"""Calls with units of both row-tile classes, which are one launch: cut into slices or whole, with the tables among the kernel's
arguments or staged, all workgroups on the chip at once or several rounds of them, against the dense oracle; the entry point
that allocates nothing gives the same bits."""
import numpy as np
import pytest

import paper_2401_06761_amd as ap
from apar_workloads import HeadConfig, draw_candidate_tree, manual_tree, mask_rows_from_parents, spec_step_qkv, step_q
from oracle import DenseThreads

from harness import assert_close, blocks_upper_bound, pool_for, replay_trace, to_dev, to_host

pytestmark = pytest.mark.gpu


# (narrow trees, wide trees, prompt, kv heads): tables with the arguments; slices; whole units
SMALL = [(1, 1, 33, 1), (2, 1, 900, 2), (4, 3, 40, 8)]
# 16-bit kernel, whole units: fewer workgroups than the 512 that the chip holds; 544; 2304
LARGE = [(12, 9, 24, 32), (32, 9, 24, 32), (24, 66, 24, 32)]
CASES = [(dtype, d, *c) for dtype, d in (("bf16", 128), ("bf16_fp8kv", 128), ("f32", 64), ("f32", 128))
         for c in SMALL + (LARGE if dtype != "f32" else [])]


@pytest.mark.parametrize("dtype,d,narrow,wide,prompt,n_kv", CASES)
def test_narrow_and_wide_trees_in_one_call(dtype, d, narrow, wide, prompt, n_kv):
    import torch

    parents, lens = [], []
    for leaves in [3] * narrow + [70] * wide:
        root = len(parents)
        parents += [-1] + [root] * leaves
        lens += [prompt + root % 16] + [1 + (5 * i) % 23 for i in range(leaves)]
    w = manual_tree(parents, lens, HeadConfig(n_kv, n_kv, d, dtype), seed=12)
    dense = DenseThreads(n_kv, n_kv, d)
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
        assert {wg[3] & 255 for wg in wgs} == {1, 2}
        if n_kv == 32:  # four narrow trees to a workgroup; no walk is long enough among the others to be cut
            walks = [wg[1] + max(wg[5 + 6 * k] for k in range(4)) for wg in wgs]
            assert len(wgs) == (narrow + 3) // 4 + wide and max(walks) <= sum(walks) * n_kv // 256 + 16
        assert_close(to_host(outs[0]), dense.decode(q, live), dtype)
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
        if n_kv == 32 or dtype == "bf16_fp8kv":
            return
        c = 2
        q, ck, cv = spec_step_qkv(w, 1, len(live), c)
        rng = np.random.default_rng(1)
        masks = np.array([mask_rows_from_parents(draw_candidate_tree(rng, c)) for _ in live], dtype=np.uint8)
        out = torch.empty_like(to_dev(q, dtype))
        ap.apar_decode_attention_spec(h, to_dev(q, dtype), to_dev(ck, dtype), to_dev(cv, dtype), torch.from_numpy(masks).cuda(), c, live, out)
        torch.cuda.synchronize()
        assert_close(to_host(out), dense.decode_spec(q, ck, cv, masks, live), dtype, "candidates")
