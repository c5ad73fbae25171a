"""Calls of two streams that share the host link: a call holds it for its host blocks only, and a call that
waits for it moves its staging blocks meanwhile.  Measured against the two calls one after the other."""
import numpy as np
import pytest

from paper_2606_14779_amd import kvpool as K

from gpu_util import say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SPEC = K.KVSpec(4, 8, 128, 16, 2, 0)   # 256 KiB blocks: 4.6 us each on the link, 0.09 us in HBM
ROOM = (401, 40000)                    # host and staging blocks of each of two requests


@pytest.fixture(scope="module")
def placed():
    """A pool with two requests, the caches, and four streams.  A process has four hardware queues, and a
    stream that shares one with the pool's own runs behind that one's work: the second call is tried on each
    of three."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = sum(ROOM)
    regions = [K.Region(k, 2 * -(-(c + 1) * SPEC.block_bytes // 4096) * 4096) for k, c in zip(("host", "staging"), ROOM)]
    with K.KVPool(regions, ROOM, SPEC) as pool:
        streams = [torch.cuda.Stream() for _ in range(4)]
        maps = [pool.place(r, n) for r in (1, 2)]
        src = torch.randint(-2**15, 2**15, (4, 2, 2 * n, 8, 16, 128), dtype=torch.int16, device="cuda")
        dst = torch.zeros_like(src)
        (sk, sv), (dk, dv) = [[[c[i].data_ptr() for c in t] for i in (0, 1)] for t in (src, dst)]
        pool.store(np.concatenate(maps), np.arange(2 * n, dtype=np.int32), 2 * n, sk, sv,
                   torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        yield pool, streams, maps, src, dst, (sk, sv), (dk, dv)
        torch.cuda.synchronize()


# (host, staging) blocks of the first and the second call, and their share of the two times' sum
@pytest.mark.parametrize("first,second,most", [
    ((1, 20000), (400, 0), 0.85),       # nearly all in HBM: the other call need not wait for it
    ((400, 200), (1, 20000), 0.85),     # a link-bound call does not hold up the other's staging blocks
    ((400, 40000), (400, 0), 0.93),     # HBM takes a little longer: the link is handed on when it is free
    ((400, 200), (400, 20000), 1.05),   # both need the link: one after the other, no slower than that
])
@pytest.mark.parametrize("op", ["retrieve", "store"])
def test_two_streams(placed, op, first, second, most):
    pool, streams, maps, src, dst, src_ptrs, dst_ptrs = placed
    n = len(maps[0])
    picks = [np.sort(np.concatenate([np.flatnonzero(m["region"] == r)[:w] for r, w in enumerate(want)]))
             for m, want in zip(maps, (first, second))]
    slots = [picks[0], n + picks[1]]

    def call(i, stream):
        getattr(pool, op)(maps[i][picks[i]].copy(), slots[i].astype(np.int32), 2 * n,
                          *(src_ptrs if op == "store" else dst_ptrs), stream.cuda_stream)

    def ms(calls):
        best = float("inf")
        for trial in range(9):
            pair = streams[0], streams[1 + trial % 3]
            torch.cuda.synchronize()
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for s in pair:
                s.wait_stream(torch.cuda.current_stream())
            for i in calls:
                call(i, pair[i])
            for s in pair:
                torch.cuda.current_stream().wait_stream(s)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        return best

    dst.zero_()
    one, two, whole = ms([0]), ms([1]), ms([0, 1])
    say("%s %s and %s: %.2f and %.2f ms, together %.2f" % (op, first, second, one, two, whole))
    assert whole < most * (one + two)
    if op == "retrieve":
        for at in slots:
            at = torch.from_numpy(at).cuda()
            assert bool((dst[:, :, at] == src[:, :, at]).all())
