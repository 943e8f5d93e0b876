"""Units whose list is cut four ways: every block is there once for its rows, the wavefronts' shares are level in full tiles
where an open tile costs two (16-bit pools) or one (fp32), and all open tiles sit with the last wavefront where they are a
quarter of the list at most."""
import numpy as np
import pytest

import paper_2401_06761_amd as ap

from harness import check_plan_covers_tables


@pytest.mark.parametrize("dtype,cost", [("bf16", 2), ("bf16_fp8kv", 2), ("f32", 1)])
@pytest.mark.parametrize("prompt,leaves", [(16 * 16, [1]), (300, [90, 33, 17, 64, 5]), (4000, [7]), (100, [15] * 12), (250, [3, 16, 32, 1, 1, 1, 1]),
                                           (16, [40, 56, 8, 24, 120, 72])])
def test_four_level_shares(dtype, cost, prompt, leaves):
    with ap.Pool(2, 2, 128, dtype, 1024, max_threads=64, dry_run=True) as pool:
        h = pool.handle
        root = ap.apar_thread_create(h)
        ap.apar_append_kv(h, root, None, None, prompt)
        live = ap.apar_fork(h, root, len(leaves))
        ap.apar_free_thread(h, root)
        for t, n in zip(live, leaves):
            ap.apar_append_kv(h, t, None, None, n)
        ap.apar_decode_attention(h, None, live, None)
        check_plan_covers_tables(h, live, 2, 1)
        wgs = np.asarray(ap.apar_last_plan_export(h, ap.APAR_PLAN_WORKGROUPS)).reshape(-1, 32)
        assert len(wgs) == 1
        wg = wgs[0]
        assert all(wg[9 + 6 * k] & 2 for k in range(4)), "one unit, cut four ways"
        tiles, full = [wg[5 + 6 * k] for k in range(4)], wg[28:32]
        n, n_full = sum(tiles), sum(full)
        n_open = n - n_full
        share = [f + cost * (t - f) for t, f in zip(tiles, full)]
        if n_full >= 3 * n // 4:
            assert all(t == f for t, f in zip(tiles[:3], full[:3]))
            # the last wavefront has more than its quarter only where the open tiles alone are more
            assert share[3] <= max(sum(share) / 4 + 1, cost * n_open)
            assert max(share[:3]) - min(share[:3]) <= 1
        else:
            assert max(share) - min(share) <= 2 * cost
