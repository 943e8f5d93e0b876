"""Appends of more blocks than fit the kernel's arguments one by one, most of them whole: by a word each, from the smallest such
call to the largest and one beyond, behind a filling block, behind a copy-on-write copy, with and without an open block at the
end, on block ids that are out of order; what the pool holds then is what the dense oracle holds."""
import pytest

import paper_2401_06761_amd as ap

from test_gpu_append_blocks import Both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16_fp8kv", 128), ("f32", 64)])
@pytest.mark.parametrize("before,rows", [(0, 16 * 121), (0, 16 * 300 + 7), (5, 16 * 130), (15, 16 * 200 + 1), (0, 16 * 956), (0, 16 * 957), (3, 16 * 952 + 13)])
def test_long_appends(dtype, d, before, rows):
    b = Both(dtype, d, n_kv=2, blocks=2400)
    scattered = [b.create(16 * (1 + k % 3)) for k in range(40)]
    for t in scattered[::2] + scattered[1::4]:  # ids come back out of order
        ap.apar_free_thread(b.h, t)
        b.dense.free(t)
        b.led.free(t)
    t = b.create(before)
    kid = b.fork(t, 1)[0] if before else b.create(0)
    b.append(t, rows)
    b.append(kid, 16 * 125 + 2)  # its filling block is copied, or written in place where the other's was
    b.check([t, kid])
