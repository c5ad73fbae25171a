"""Calls captured into a HIP graph: small ones, and allocation-free retrieves of any size, whose work
lists both travel in kernel arguments.  Every replay is checked against the eager result, with eager calls
of the library between replays; a call that would upload its list is refused."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from kvgen import workloads
from paper_2606_14779_amd import kvpool as K

from gpu_util import check_full, make_run, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


def _run(n):
    rng = np.random.default_rng(n)
    shape = workloads.KVShape("captured", 4, 2, 64)
    regions = [workloads.RegionSpec("host", 1, 0), workloads.RegionSpec("staging", 2)]
    req = workloads.RequestSpec(1, n, n, rng.permutation(n + 9)[:n].astype(np.int32),
                                rng.permutation(n + 9)[:n].astype(np.int32))
    wl = workloads.Workload(0, "captured", 93, shape, 0, regions, [req], n + 9, n + 9)
    workloads._size_regions(wl.regions, [n], shape.block_bytes)
    return make_run(wl)


@pytest.mark.parametrize("call,n", [("retrieve", 20), ("store", 20), ("retrieve_noalloc", 20),
                                    ("retrieve_noalloc", 400)])
def test_replays_equal_the_eager_call(call, n):
    say("case", call, n)
    run = _run(n)
    try:
        host = run.setup(keep_host=True)
        q = run.wl.requests[0]
        store = call == "store"
        cache = run.src if store else run.dst
        table, slots = (q.src_slots, run.wl.src_num_slots) if store else (q.dst_slots, run.wl.dst_num_slots)
        k, v = run.layer_ptrs(cache)

        def enqueue():
            getattr(run.pool, call)(run.maps[1], table, slots, k, v, torch.cuda.current_stream().cuda_stream)

        enqueue()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            enqueue()
        small = run.maps[1][:3]
        for i in range(4):
            run.fill_dst()
            if store:
                run.src.add_(1)   # other contents each time: the replay has to store these
                host += np.uint16(1)
            g.replay()
            if store:
                run.retrieve_all()
            torch.cuda.synchronize()
            check_full(run.wl, run, host)
            # eager calls between the replays, on this and another stream; they land where they did
            run.pool.retrieve(small, q.dst_slots[:3], run.wl.dst_num_slots, *run.layer_ptrs(run.dst),
                              torch.cuda.current_stream().cuda_stream)
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            run.pool.retrieve(small, q.dst_slots[:3], run.wl.dst_num_slots, *run.layer_ptrs(run.dst), side.cuda_stream)
            torch.cuda.synchronize()
        run.pool.release(1)
    finally:
        run.close()


@pytest.mark.parametrize("layers,heads,head_dim,layout", [(4, 2, 64, 0), (4, 2, 64, 1), (150, 1, 8, 0), (400, 1, 8, 1)])
def test_captured_lists_are_not_shared(layers, heads, head_dim, layout):
    """Two allocation-free calls with lists too large for one launch's arguments, captured into one graph,
    and larger and smaller eager ones between capture and replay, on this and another pool: every replay
    writes what the two calls named, and nothing else.  With 150 layers the engine pointers take most of
    the arguments, with 400 they exceed them."""
    rng = np.random.default_rng(layers)
    shape = workloads.KVShape("captured", layers, heads, head_dim)
    n = 420
    regions = [workloads.RegionSpec("host", 1, 0), workloads.RegionSpec("staging", 2)]
    say("case captured lists", layers, heads, head_dim, layout)

    def one():
        req = workloads.RequestSpec(1, n, n, rng.permutation(n + 9)[:n].astype(np.int32),
                                    rng.permutation(n + 9)[:n].astype(np.int32))
        wl = workloads.Workload(0, "captured", 95, shape, layout, list(regions), [req], n + 9, n + 9)
        workloads._size_regions(wl.regions, [n], shape.block_bytes)
        return make_run(wl)

    run, other = one(), one()
    try:
        host = run.setup(keep_host=True)
        other.setup()
        q, m = run.wl.requests[0], run.maps[1]
        k, v = run.layer_ptrs(run.dst)

        def eager(r, count):
            r.pool.retrieve_noalloc(r.maps[1][:count], r.wl.requests[0].dst_slots[::-1][:count].copy(),
                                    r.wl.dst_num_slots, *r.layer_ptrs(r.dst), torch.cuda.current_stream().cuda_stream)

        eager(run, n)   # both halves of the scratch are in use before the capture too
        eager(run, 300)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for part in (slice(0, 200), slice(200, n)):
                run.pool.retrieve_noalloc(m[part], q.dst_slots[part].copy(), run.wl.dst_num_slots, k, v,
                                          torch.cuda.current_stream().cuda_stream)
        for count in (n, 300, 250):
            eager(run, count)
            eager(other, count)
            torch.cuda.synchronize()
            run.fill_dst()
            g.replay()
            torch.cuda.synchronize()
            check_full(run.wl, run, host)
        run.pool.release(1)
    finally:
        run.close()
        other.close()


def test_a_call_with_an_uploaded_list_is_refused():
    run = _run(400)
    try:
        run.setup()
        q = run.wl.requests[0]
        k, v = run.layer_ptrs(run.dst)
        x = torch.zeros(16, device="cuda")
        g = torch.cuda.CUDAGraph()
        codes = []
        with torch.cuda.graph(g):
            x.add_(1)
            try:
                run.pool.retrieve(run.maps[1], q.dst_slots, run.wl.dst_num_slots, k, v,
                                  torch.cuda.current_stream().cuda_stream)
            except K.KVPoolError as e:
                codes.append(e.name)
        assert codes == ["HIP"]
        run.fill_dst()
        before = run.dst.clone()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(run.dst, before)   # nothing of the refused call is in the graph
    finally:
        run.close()


@pytest.mark.parametrize("thread", ["same", "other"])
@pytest.mark.parametrize("mode", ["global", "thread_local", "relaxed"])
def test_small_calls_beside_a_capture(mode, thread):
    """Eager small calls on one stream while another is being captured, from the capturing thread and from
    another, with earlier calls in flight: they run, and the capture goes on unharmed."""
    run = _run(20)
    pool = ThreadPoolExecutor(1)
    try:
        host = run.setup(keep_host=True)
        q = run.wl.requests[0]
        side = torch.cuda.Stream()
        dst, src = run.layer_ptrs(run.dst), run.layer_ptrs(run.src)
        x = torch.zeros(16, device="cuda")
        torch.cuda.synchronize()

        def calls():
            for i in range(40):   # more than the events that a pool starts with
                run.pool.store(run.maps[1], q.src_slots, run.wl.src_num_slots, *src, side.cuda_stream)
                run.pool.retrieve(run.maps[1], q.dst_slots, run.wl.dst_num_slots, *dst, side.cuda_stream)
                run.pool.retrieve_noalloc(run.maps[1], q.dst_slots, run.wl.dst_num_slots, *dst, side.cuda_stream)

        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, capture_error_mode=mode):
            x.add_(1)
            calls() if thread == "same" else pool.submit(calls).result()
            x.add_(1)
        torch.cuda.synchronize()
        check_full(run.wl, run, host)
        for i in range(3):
            g.replay()
            torch.cuda.synchronize()
            assert bool((x == 2 * i + 2).all())
        run.pool.release(1)
    finally:
        pool.shutdown()
        run.close()


def test_thousands_of_calls_in_flight():
    """More calls than completion events exist at first, over three streams; each request's release
    waits for its own."""
    run = _run(6)
    try:
        host = run.setup(keep_host=True)
        streams = [torch.cuda.Stream() for _ in range(3)]
        for s in streams:
            s.wait_stream(torch.cuda.current_stream())
        for i in range(3000):
            run.retrieve(run.wl.requests[0], streams[i % 3])
        torch.cuda.synchronize()
        check_full(run.wl, run, host)
        run.pool.release(1)
    finally:
        run.close()
