"""Which kernels a call launches, by the runtime's own trace: one launch for both region classes, or one per
class where that is asked for or the flags need it.  Results are checked against the oracle in either form."""
import numpy as np
import pytest

from kvgen import workloads
from paper_2606_14779_amd import kvpool as K

from gpu_util import check_full, make_run, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NT = K.LAUNCH_NT_LOAD | K.LAUNCH_NT_STORE
BOTH, EACH = ["both_regions_copy"], ["host_region_copy", "staging_region_copy"]


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


def _kernels(call):
    """Names of the library's copy kernels that ran in the call, sorted, without the list's upload."""
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    names = [e.name for e in prof.events() if "kvp::" in e.name]
    return sorted(n.split("kvp::")[1].split("<")[0].split("(")[0] for n in names if "list_copy" not in n)


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("host_flags,staging_flags,timed,expect", [
    (0, NT, False, BOTH),
    (0, NT, True, EACH),
    (K.LAUNCH_XCD, NT, False, EACH),
    (K.LAUNCH_CHUNK_MAJOR, NT, False, EACH),
    (K.LAUNCH_TILE, NT, False, EACH),
    (K.LAUNCH_SPLIT2, NT | K.LAUNCH_XCD | K.LAUNCH_TILE, False, BOTH),   # the staging class ignores those
    (0, K.LAUNCH_NT_LOAD, False, EACH),
    (0, K.LAUNCH_NT_STORE, False, None),   # its loads keep their lines in a token-major pool's one launch only
])
def test_kernels_of_a_call(host_flags, staging_flags, timed, expect, layout):
    n = 300   # more than the kernel arguments hold
    rng = np.random.default_rng(n)
    shape = workloads.KVShape("dispatch", 4, 2, 64)
    regions = [workloads.RegionSpec("host", 1, 0), workloads.RegionSpec("staging", 2)]
    req = workloads.RequestSpec(1, n, n, rng.permutation(n + 9)[:n].astype(np.int32),
                                rng.permutation(n + 9)[:n].astype(np.int32))
    wl = workloads.Workload(0, "dispatch", 93, shape, layout, regions, [req], n + 9, n + 9)
    workloads._size_regions(wl.regions, [n], shape.block_bytes)
    say("case", host_flags, staging_flags, timed, layout)
    run = make_run(wl)
    try:
        for op in (K.OP_RETRIEVE, K.OP_STORE):
            run.pool.set_launch(K.CLASS_HOST, op, 0, host_flags)
            run.pool.set_launch(K.CLASS_STAGING, op, 0, staging_flags)
        host = run.setup(keep_host=True)
        run.retrieve_all()
        torch.cuda.synchronize()
        run.pool.set_timing(timed)
        names = _kernels(run.retrieve_all)
        assert names == ((BOTH if layout else EACH) if expect is None else expect)
        assert _kernels(run.store_all) == names
        check_full(wl, run, host)
    finally:
        run.close()
