"""Calls of several host threads on hipStreamPerThread, one handle that names another stream in every
thread: data ordering (a retrieve after a store, a store after a retrieve) and release hold across them."""
import time
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from kvgen import workloads

from gpu_util import make_run, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PER_THREAD = 2   # hipStreamPerThread


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


def _run(n):
    """n blocks of 256 KiB in one host region: a call of all of them holds the link for 4.6 us a block."""
    rng = np.random.default_rng(n)
    shape = workloads.KVShape("threads", 4, 8, 128)
    req = workloads.RequestSpec(1, n, n, rng.permutation(n)[:n].astype(np.int32), rng.permutation(n)[:n].astype(np.int32))
    wl = workloads.Workload(0, "threads", 97, shape, 0, [workloads.RegionSpec("host", 1, 0)], [req], n, n)
    workloads._size_regions(wl.regions, [n], shape.block_bytes)
    return make_run(wl)


@pytest.fixture
def threads():
    """Two host threads, each with a stream of its own behind that handle; they outlive all work on it (a
    thread that ends takes its stream with it)."""
    a, b = ThreadPoolExecutor(1), ThreadPoolExecutor(1)
    yield lambda f: a.submit(f).result(), lambda f: b.submit(f).result()
    torch.cuda.synchronize()
    a.shutdown()
    b.shutdown()


def _moved(run):
    q = run.wl.requests[0]
    src = run.src[:, :, torch.from_numpy(q.src_slots.astype(np.int64)).cuda()]
    return src, run.dst[:, :, torch.from_numpy(q.dst_slots.astype(np.int64)).cuda()]


def test_data_order_between_threads(threads):
    in_a, in_b = threads
    run = _run(400)
    try:
        run.setup()
        q = run.wl.requests[0]
        m = run.maps[1]
        src_ptrs, dst_ptrs = run.layer_ptrs(run.src), run.layer_ptrs(run.dst)

        def store():
            run.pool.store(m, q.src_slots, run.wl.src_num_slots, *src_ptrs, PER_THREAD)

        def retrieve():
            run.pool.retrieve(m, q.dst_slots, run.wl.dst_num_slots, *dst_ptrs, PER_THREAD)

        in_a(retrieve)
        torch.cuda.synchronize()
        for i in range(3):
            say("round", i)
            run.src.add_(1)
            run.fill_dst()
            torch.cuda.synchronize()
            in_a(store)      # a retrieve right behind it reads the new contents
            in_b(retrieve)
            torch.cuda.synchronize()
            src, dst = _moved(run)
            assert bool((src == dst).all())
            run.src.add_(1)
            run.fill_dst()
            torch.cuda.synchronize()
            in_a(retrieve)   # a store right behind it changes nothing of what it reads
            in_b(store)
            torch.cuda.synchronize()
            src, dst = _moved(run)
            assert bool((src - 1 == dst).all())
    finally:
        run.close()


def test_release_waits_for_every_thread(threads):
    in_a, in_b = threads
    run = _run(4000)   # 1 GiB, over 18 ms on the link
    try:
        run.setup()
        q = run.wl.requests[0]
        m = run.maps[1]
        ptrs = run.layer_ptrs(run.dst)
        torch.cuda.synchronize()
        done = torch.cuda.Event()

        def whole():
            run.pool.retrieve(m, q.dst_slots, run.wl.dst_num_slots, *ptrs, PER_THREAD)
            done.record(torch.cuda.ExternalStream(PER_THREAD))

        def one():
            run.pool.retrieve(m[:1], q.dst_slots[:1], run.wl.dst_num_slots, *ptrs, PER_THREAD)

        in_a(whole)
        in_b(one)
        run.pool.release(1)
        t0 = time.perf_counter()
        done.synchronize()
        assert time.perf_counter() - t0 < 5e-3   # the long retrieve was over when release returned
    finally:
        run.close()
