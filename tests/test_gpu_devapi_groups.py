"""GPU parity: device API calls from user kernels whose work-groups are not
whole wavefronts, down to one thread, checked byte for byte."""
import ctypes

import numpy as np
import pytest

import oracle
import workload as W
from tests.gpu_helpers import assert_no_device_errors, download, heap, torch, upload, user_lib

pytestmark = pytest.mark.gpu

THREADS = [1, 2, 16, 32, 48, 96]   # below a wavefront, and one and a half


@pytest.mark.parametrize("nwgs", [1, 3])   # the _wg and the _grid calls
@pytest.mark.parametrize("wg", THREADS)
def test_put_and_get_by_any_work_group(wg, nwgs):
    """Blocks around a vector and a batch, for destinations and sources on and
    off the 16-byte boundaries: the block and nothing else is written."""
    lib = user_lib()
    npes = 3
    with heap(npes, 1 << 20) as v:
        src, dst = v.malloc(16384), v.malloc(16384)
        so, do = v.offset(src), v.offset(dst)
        init = W.heap_fill(0x6A0 + wg, npes, do + 16384)
        for get in (0, 1):
            for n in (1, 15, 16, 17, 33, 64, 250, 4099):
                for a, b in ((0, 0), (0, 1), (3, 8), (5, 15)):
                    upload(init)
                    assert lib.usertest_move(v.device_ctx(), npes, get, src + a, dst + b, n, nwgs, wg, None) == 0
                    torch().cuda.synchronize()
                    ref = init.copy()
                    for p in range(npes):
                        q = (p + 1) % npes
                        s, d = (q, p) if get else (p, q)
                        ref[d, do + b:do + b + n] = init[s, so + a:so + a + n]
                    assert np.array_equal(download(init.shape[1]), ref), (get, n, a, b)
        assert_no_device_errors()


@pytest.mark.parametrize("nwgs", [1, 16])
@pytest.mark.parametrize("wg", [1, 16, 32, 48, 96])
@pytest.mark.parametrize("kind", [0, 1, 2])   # broadcast, fcollect, alltoall
def test_movement_collectives_by_any_work_group(kind, wg, nwgs):
    """Blocks on both sides of what 16 and 32 lanes move in a pass (1, 2, 4
    KiB), and of the size where fcollect leaves the pairs (16 KiB)."""
    lib = user_lib()
    npes = 3
    t = torch()
    with heap(npes, 1 << 20) as v:
        team = v.team_device(v.TEAM_WORLD)
        src, dst = v.malloc(npes * 20480), v.malloc(npes * 20480)
        so, do = v.offset(src), v.offset(dst)
        init = W.heap_fill(0x6B0 + wg, npes, do + npes * 20480)
        status = t.zeros(npes * nwgs, dtype=t.int32, device="cuda")
        for n in (1, 24, 1025, 2049, 4097, 9000, 16385):
            for a, b in ((0, 0), (3, 5)):
                upload(init)
                assert lib.usertest_collective_any(v.device_ctx(), ctypes.byref(team), kind, dst + b, src + a, n, 1,
                                                   nwgs, wg, status.data_ptr(), None) == 0
                t.cuda.synchronize()
                assert (status.cpu().numpy() == 0).all()
                ref = init.copy()
                if kind == 0:
                    oracle.broadcast(ref, do + b, so + a, n, 1)
                elif kind == 1:
                    oracle.fcollect(ref, do + b, so + a, n)
                else:
                    oracle.alltoall(ref, do + b, so + a, n)
                assert np.array_equal(download(init.shape[1]), ref), (n, a, b)
        assert_no_device_errors()
