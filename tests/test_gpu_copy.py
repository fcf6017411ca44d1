"""The copy engine at its edges: every pair of source and destination
alignments modulo 16 at the lengths where a path or a batch ends."""
import numpy as np
import pytest

import workload as W
from tests.gpu_helpers import assert_no_device_errors, device_array, download, heap, upload

pytestmark = pytest.mark.gpu

# Around 16 bytes (vectors begin), a wavefront's and a work-group's pass (64
# and 128 lanes), and a full batch of four and eight vectors per lane.
SIZES = [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 250, 1023, 1024, 1040, 2063, 4095, 4112, 8209]


@pytest.mark.parametrize("flags", [0, 3])   # temporal four deep; nontemporal eight deep
@pytest.mark.parametrize("scope", [W.SCOPE_THREAD, W.SCOPE_WAVE, W.SCOPE_WG, W.SCOPE_GRID])
def test_every_alignment_pair(scope, flags):
    """Sixteen messages whose sources step through the alignments, for each
    destination alignment: bytes equal the numpy move, and the gaps between
    messages keep theirs."""
    npes, area = 2, 16 * 16 * (max(SIZES) + 64)
    with heap(npes, 2 * area + (1 << 20)) as v:
        base = v.offset(v.malloc(2 * area + 4096))
        init = W.heap_fill(0xA11 + scope, npes, base + 2 * area + 4096)
        tgt = device_array(np.array([1, 0], dtype=np.int32))
        launch = v.launch_cfg(wgs_per_pe=2, wg_size=128, flags=flags)
        for n in SIZES:
            pitch = (n + 15) // 16 * 16 + 32        # a message's room: its step keeps the destination's alignment
            upload(init)
            ref = init.copy()
            for d in range(16):
                so, do = base, base + area + d * 16 * pitch + d
                v.rma_pattern(W.OP_PUT, scope, tgt, so, do, n, 16, pitch + 1, pitch, launch=launch)
                for j in range(16):
                    for p in range(npes):
                        ref[1 - p, do + j * pitch:do + j * pitch + n] = \
                            init[p, so + j * (pitch + 1):so + j * (pitch + 1) + n]
            assert np.array_equal(download(init.shape[1]), ref), n
        assert_no_device_errors()


@pytest.mark.parametrize("scope", [W.SCOPE_THREAD, W.SCOPE_WAVE, W.SCOPE_WG, W.SCOPE_GRID])
def test_runs_of_messages(scope):
    """Packed and spaced runs, with more, as many and fewer messages than
    units, around a unit's batch (64, 128 or 384 lanes of four vectors)."""
    npes, area = 3, 1 << 20
    with heap(npes, 4 * area) as v:
        base = v.offset(v.malloc(2 * area + 4096))
        init = W.heap_fill(0xA22 + scope, npes, base + 2 * area + 4096)
        tgt = device_array(np.array([1, 2, 0], dtype=np.int32))
        launch = v.launch_cfg(wgs_per_pe=3, wg_size=128)
        for n in (1, 7, 8, 13, 16, 40, 1000, 4096, 4097, 8192, 24576, 32768, 40000, 98304):
            for count in (1, 2, 7, 100):
                for sgap, dgap, ss, ds in ((0, 0, 0, 0), (0, 0, 5, 0), (0, 16, 0, 0), (3, 9, 1, 2), (-n, 0, 4, 4)):
                    if count * (n + 16) > area:
                        continue
                    upload(init)
                    so, do = base + ss, base + area + ds
                    v.rma_pattern(W.OP_GET, scope, tgt, so, do, n, count, n + sgap, n + dgap, launch=launch)
                    ref = init.copy()
                    for p in range(npes):
                        q = (p + 1) % npes
                        for j in range(count):
                            s, d = so + j * (n + sgap), do + j * (n + dgap)
                            ref[p, d:d + n] = init[q, s:s + n]
                    assert np.array_equal(download(init.shape[1]), ref), (n, count, sgap, dgap, ss, ds)
        assert_no_device_errors()
