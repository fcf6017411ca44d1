"""GPU parity: device API calls from user kernels whose work-groups are not
whole wavefronts, down to one thread, checked byte for byte."""
import numpy as np
import pytest

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
