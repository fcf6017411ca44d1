"""Reductions split over wavefronts, around the counts where a work-group's
task changes from one tile of 64 vectors to a step of several and where the
split form ends."""
import numpy as np
import pytest

import oracle
import workload as W
from tests.gpu_helpers import assert_no_device_errors, download, heap, torch, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("npes,sixteenths", [(24, 7), (31, 7), (32, 8), (40, 8)])
@pytest.mark.parametrize("dt", [oracle.DT_INT64, oracle.DT_FP32, oracle.DT_BF16])
def test_reductions_around_the_step_edges(dt, npes, sixteenths):
    """Bit-exact against the oracle, nothing else written."""
    es = {oracle.DT_INT64: 8, oracle.DT_FP32: 4, oracle.DT_BF16: 2}[dt]
    gen = {oracle.DT_INT64: W.coll_i64, oracle.DT_FP32: W.coll_f32, oracle.DT_BF16: W.coll_bf16}[dt]
    cus = torch().cuda.get_device_properties(0).multi_processor_count
    one, limit = 64 * (cus // npes * npes), sixteenths * cus * 16
    with heap(npes, 2 << 20) as v:
        room = (limit + 2) * 16
        src, dst = v.malloc(room), v.malloc(room)
        so, do = v.offset(src), v.offset(dst)
        for nvec in (65, 129, one, one + 1, limit, limit + 1):
            n = nvec * 16 // es + 1
            init = W.heap_fill(0xE8, npes, do + room)
            for p in range(npes):
                init[p, so:so + n * es] = np.ascontiguousarray(gen(0xE7, p, n)).view(np.uint8)
            upload(init)
            v.reduce(dt, oracle.RO_SUM, dst, src, n)
            ref = init.copy()
            oracle.reduce(ref, dt, oracle.RO_SUM, do, so, n)
            assert np.array_equal(download(do + room), ref), nvec
        assert_no_device_errors()
