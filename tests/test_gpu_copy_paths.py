"""The copy engine as user kernels and batches call it (one lane, a wavefront
or a work-group per message): every pair of source and destination alignments
modulo 16, at the lengths where its paths change."""
import numpy as np
import pytest

import workload as W
from tests.gpu_helpers import assert_no_device_errors, device_array, download, heap, torch, upload, user_lib

pytestmark = pytest.mark.gpu

# One lane: pieces of 1 to 16 bytes, two of them up to 32, four vectors at a
# time.  Lanes together: below 16 bytes; one piece per lane up to 16 times
# their number; two, then four per lane; a batch and its remainder.
SIZES = {
    W.SCOPE_THREAD: [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 80, 112, 250],
    W.SCOPE_WAVE: [1, 15, 16, 17, 31, 250, 1008, 1009, 1024, 1025, 1041, 2047, 2049, 4079, 4095, 4096, 4097, 4112, 6200],
    W.SCOPE_WG: [8, 16, 1500, 2033, 2048, 2049, 4097, 8191, 8192, 8193, 8208],   # by 128 lanes
}
NPES = 2


def _layout(sizes, base):
    """(source, destination, bytes) of a message per length and alignment
    pair, none overlapping another; the bytes of heap they take."""
    ops, so = [], base
    for n in sizes:
        for a in range(16):
            for b in range(16):
                ops.append([so + a, 0, n])
                so += n + 32 + 15 & ~15
    room = so - base
    for op, d in zip(ops, range(len(ops))):
        op[1] = op[0] - base - (op[0] & 15) + base + room + d % 16   # b = d mod 16
    return np.array(ops, dtype=np.uint64), 2 * room


def _expect(init, ops, get):
    ref = init.copy()
    for p in range(NPES):
        s, d = (1 - p, p) if get else (p, 1 - p)
        for so, do, n in ops.astype(np.int64):
            ref[d, do:do + n] = init[s, so:so + n]
    return ref


@pytest.mark.parametrize("get", [0, 1])
@pytest.mark.parametrize("scope", [W.SCOPE_THREAD, W.SCOPE_WAVE, W.SCOPE_WG])
def test_user_kernels_at_every_alignment_pair(scope, get):
    lib = user_lib()
    with heap(NPES, 64 << 20) as v:
        base = v.offset(v.malloc(48 << 20))
        ops, room = _layout(SIZES[scope], base)
        assert room < 48 << 20
        init = W.heap_fill(0xB0 + scope, NPES, base + room)
        upload(init)
        table = device_array(ops.view(np.int64))
        assert lib.usertest_moves(v.device_ctx(), NPES, scope, get, table.data_ptr(), len(ops), 128, None) == 0
        torch().cuda.synchronize()
        assert np.array_equal(download(init.shape[1]), _expect(init, ops, get))
        assert_no_device_errors()


@pytest.mark.parametrize("get", [0, 1])
@pytest.mark.parametrize("scope", [W.SCOPE_THREAD, W.SCOPE_WAVE, W.SCOPE_WG])
def test_batches_at_every_alignment_pair(scope, get):
    """The same messages as operations of a plan and of a device table."""
    with heap(NPES, 64 << 20) as v:
        base = v.offset(v.malloc(48 << 20))
        ops, room = _layout(SIZES[scope], base)
        init = W.heap_fill(0xB8 + scope, NPES, base + room)
        ref = _expect(init, ops, get)
        op = W.OP_GET if get else W.OP_PUT
        descs = W.descs([(op, scope, 0, p, 1 - p, W.NO_RESULT, int(so), int(do), int(n), 0, 0)
                         for p in range(NPES) for so, do, n in ops])
        tune = v.default_tune()
        tune.wg_size = 128
        plan = v.Plan(descs, tune=tune)
        table = device_array(np.ascontiguousarray(descs).view(np.uint8).copy())
        for run in (plan.launch_fused, lambda: v.launch_batch(table, len(descs))):
            upload(init)
            run()
            torch().cuda.synchronize()
            assert np.array_equal(download(init.shape[1]), ref)
        plan.destroy()
        assert_no_device_errors()
