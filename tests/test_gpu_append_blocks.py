"""Appends write a block in one pass (copy-on-write rows, new rows, matrix-core order once full): every start and end slot,
threads listed in several places, source-row lists, calls with more blocks than go along with the kernel's arguments,
and a shared block that its last holder fills in the call that others copy it in."""
import numpy as np
import pytest

import paper_2401_06761_amd as ap
from apar_workloads import quantise
from oracle import BlockLedger, DenseThreads

from harness import books_equal, to_dev, to_host

pytestmark = pytest.mark.gpu


class Both:
    """The library and the dense oracle under the same operations; rows are compared through apar_read_kv_rows."""

    def __init__(self, dtype, d, n_kv=3, blocks=4000):
        self.dtype, self.d, self.n_kv = dtype, d, n_kv
        self.pool = ap.Pool(n_kv, n_kv, d, dtype, blocks, max_threads=4096)
        ap.apar_set_write_checks(self.pool.handle, True)
        self.pool.kv.fill_(0xFF)
        self.h = self.pool.handle
        self.dense, self.led = DenseThreads(n_kv, n_kv, d), BlockLedger(blocks)
        self.rng = np.random.default_rng(d)

    def rows(self, n):
        return [quantise(self.rng.standard_normal((n, self.n_kv, self.d)).astype(np.float32), self.dtype, kv=True) for _ in "kv"]

    def create(self, n):
        t = ap.apar_thread_create(self.h)
        assert t == self.dense.create() == self.led.create()
        if n:
            self.append(t, n)
        return t

    def append(self, t, n):
        k, v = self.rows(n)
        ap.apar_append_kv(self.h, t, to_dev(k, self.dtype), to_dev(v, self.dtype), n)
        self.dense.append(t, k, v)
        self.led.append(t, n)

    def fork(self, t, n):
        kids = ap.apar_fork(self.h, t, n)
        assert list(kids) == list(self.dense.fork(t, n)) == list(self.led.fork(t, n))
        return kids

    def batch(self, threads, src=None):
        k, v = self.rows(len(threads) if src is None else max(src) + 1)
        kd, vd = to_dev(k, self.dtype), to_dev(v, self.dtype)
        if src is None:
            ap.apar_append_kv_batch(self.h, threads, kd, vd)
        else:
            ap.apar_append_kv_gather(self.h, threads, src, kd, vd)
        for i, t in enumerate(threads):
            r = i if src is None else src[i]
            self.dense.append(t, k[r:r + 1], v[r:r + 1])
        self.led.append_batch(threads)

    def check(self, threads):
        import torch

        books_equal(self.h, self.led, check_blocks=range(64))
        for t in threads:
            L = self.dense.length(t)
            k = torch.empty((L, self.n_kv, self.d), dtype=self.pool.torch_dtype, device="cuda:0")
            v = torch.empty_like(k)
            ap.apar_read_kv_rows(self.h, t, 0, L, k, v)
            torch.cuda.synchronize()
            K, V = self.dense.rows(t)
            assert np.array_equal(to_host(k), K) and np.array_equal(to_host(v), V), f"thread {t}"


KINDS = [("f32", 64), ("f32", 128), ("bf16", 128), ("bf16_fp8kv", 128)]


@pytest.mark.parametrize("dtype,d", KINDS)
def test_every_start_and_end_slot(dtype, d):
    b = Both(dtype, d)
    threads = []
    for start in (0, 1, 7, 15, 16):
        for n in (1, 2, 8, 9, 15, 16, 17, 40):
            t = b.create(start)
            b.append(t, n)
            threads.append(t)
    b.check(threads)
    b.append(threads[0], 16 * 130 + 5)  # more blocks than the kernel's arguments carry
    b.check(threads[:2])


@pytest.mark.parametrize("dtype,d", KINDS)
@pytest.mark.parametrize("tail", [1, 13, 14, 15])
def test_shared_tails_copied_filled_and_sealed_in_one_call(dtype, d, tail):
    b = Both(dtype, d)
    t = b.create(16 + tail)
    family = [t] + list(b.fork(t, 3))
    other = b.create(5)
    # the last one listed holds the shared tail alone by then and writes in place; with several rows each it fills it
    b.batch(family)
    b.check(family)
    kids = list(b.fork(family[1], 2))
    listed = [family[1], kids[0], other, kids[1], kids[0], kids[1], kids[0], kids[1], kids[1]]
    b.batch(listed)
    b.check(family + kids + [other])
    again = list(b.fork(other, 2))
    b.batch([again[0], other, again[1], other, again[0]], src=[4, 0, 9, 2, 2])
    b.check(again + [other])


@pytest.mark.parametrize("dtype,d", KINDS)
def test_many_threads_beyond_the_kernel_arguments(dtype, d):
    b = Both(dtype, d)
    root = b.create(30)
    kids = list(b.fork(root, 300))
    for step in range(3):  # copies of the shared tail, then sealing, then fresh blocks
        b.batch(kids if step else kids[::-1])
    order = [int(x) for x in b.rng.permutation(kids)]
    b.batch(order, src=[int(x) for x in b.rng.integers(0, 50, size=len(order) - 1)] + [50])
    b.check(kids[::17] + [root])
