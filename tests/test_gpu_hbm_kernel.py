"""GPU parity of the HBM copy body (staging regions) at the edges of its units and orders: chunks of
one vector up to a few units, with and without a partial last unit; launches around and past a whole
set of per-die runs of workgroups; the last chunk group short; explicit grids smaller than the work;
work items sorted by slot over one and two digits.  Bit for bit against the CPU oracle.
"""
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


def _workload(shape, n, slots, layout):
    rng = np.random.default_rng(n + slots)
    regions = [workloads.RegionSpec("staging", 3), workloads.RegionSpec("host", 1, 0), workloads.RegionSpec("staging", 2)]
    req = workloads.RequestSpec(1, n, n, rng.permutation(slots)[:n].astype(np.int32),
                                rng.permutation(slots)[:n].astype(np.int32))
    wl = workloads.Workload(0, "hbm-edges", 91, shape, layout, regions, [req], slots, slots)
    workloads._size_regions(wl.regions, [n], shape.block_bytes)
    return wl


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("upload", [False, True])
@pytest.mark.parametrize("layers,heads,head_dim,tokens,n,slots,grid", [
    (1, 1, 8, 1, 1, 1, 0),         # a chunk of one 16-byte vector, one block
    (3, 1, 8, 63, 70, 75, 0),      # 1008 B: the only unit is one vector short; 6 chunks in groups of 4
    (3, 1, 64, 8, 70, 75, 0),      # 1024 B: exactly one unit
    (3, 5, 8, 13, 70, 2100, 0),    # 1040 B: a last unit of one vector; slots over two digits
    (1, 3, 40, 16, 65, 66, 2),     # 3840 B, 80-byte rows; a grid that has to loop
    (2, 2, 64, 16, 819, 830, 0),   # 4096 B: over 2048 workgroups, with a rest
    (2, 2, 64, 16, 819, 830, 24),  # the same, looping
    (5, 4, 24, 16, 700, 4099, 0),  # 3072 B: 10 chunks, two digits
])
def test_edges(layers, heads, head_dim, tokens, n, slots, grid, upload, layout):
    shape = workloads.KVShape("edges", layers, heads, head_dim, tokens)
    say("case", layers, heads, head_dim, tokens, n, slots, grid, upload, layout)
    run = make_run(_workload(shape, n, slots, layout))
    try:
        for op in (K.OP_RETRIEVE, K.OP_STORE):
            flags = K.LAUNCH_NT_LOAD | K.LAUNCH_NT_STORE | (K.LAUNCH_UPLOAD if upload else 0)
            run.pool.set_launch(K.CLASS_STAGING, op, grid, flags)
        host = run.setup(keep_host=True)
        run.retrieve_all()
        torch.cuda.synchronize()
        check_full(run.wl, run, host)
    finally:
        run.close()


def test_store_of_one_slot_into_many_blocks():
    """A store may name a source slot twice (only the pool blocks have to be distinct)."""
    shape = workloads.KVShape("edges", 2, 2, 64)
    wl = _workload(shape, 96, 100, 0)
    q = wl.requests[0]
    q.src_slots[:] = q.src_slots[np.arange(96) // 3]
    run = make_run(wl)
    try:
        run.src.copy_(torch.randint(-2**15, 2**15, run.src.shape, dtype=torch.int16, device="cuda"))
        run.fill_dst()
        run.place_all()
        run.store_all()
        run.retrieve_all()
        torch.cuda.synchronize()
        got = run.dst[:, :, torch.from_numpy(q.dst_slots.astype(np.int64)).cuda()]
        assert torch.equal(got, run.src[:, :, torch.from_numpy(q.src_slots.astype(np.int64)).cuda()])
    finally:
        run.close()


@pytest.mark.parametrize("vectors", [1, 255, 256, 257, 1024 * 5 + 3])
@pytest.mark.parametrize("form", [0, K.LAUNCH_SPLIT2, K.LAUNCH_TILE])
@pytest.mark.parametrize("hints", [0, K.LAUNCH_NT_LOAD, K.LAUNCH_NT_STORE, K.LAUNCH_NT_LOAD | K.LAUNCH_NT_STORE])
def test_probe_copies(vectors, form, hints):
    """The probe copy in tiles of 8, 4 and 1 vectors per lane: exactly its bytes, in every form."""
    src = torch.randint(-2**31, 2**31, (vectors * 4 + 8,), dtype=torch.int32, device="cuda")
    for grid in (0, 1, 3):
        dst = torch.zeros_like(src)
        K.probe_copy_kernel(dst.data_ptr(), src.data_ptr(), vectors * 16, grid, form | hints,
                            torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(dst[:-8], src[:-8]) and not bool(dst[-8:].any())
