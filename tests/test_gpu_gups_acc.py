"""The accumulator of random updates without fetched values: the XOR of the
values that the words held, determined where no word is updated twice."""
import numpy as np
import pytest

import workload as W
from tests.gpu_helpers import assert_no_device_errors, heap, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("explicit", [False, True])
@pytest.mark.parametrize("nupd", [1, 63, 65, 256, 257, 3000])   # within a wavefront, across them, across work-groups
def test_accumulator_without_fetched_values(nupd, explicit):
    npes, log2_table = 4, 24
    words = 1 << (log2_table - 2)
    base = next(b for b in range(W.SEED_GUPS, W.SEED_GUPS + 100)
                if len(np.unique(W.gups_updates(b, 0, nupd, log2_table, add_every=3)[0])) == nupd)
    idx = W.gups_updates(base, 0, nupd, log2_table, add_every=3)[0].astype(np.int64)
    with heap(npes, 8 * words) as v:
        t = torch()
        t.manual_seed(nupd)
        table = v.heap_view()[:, :8 * words].view(t.int64)
        table.copy_(t.randint(-2**62, 2**62, (npes, words), device="cuda"))
        want = np.bitwise_xor.reduce(table.cpu().numpy().reshape(-1)[idx])
        acc = t.zeros(1, dtype=t.int64, device="cuda")
        launch = v.Launch(3, 0, 0, 0, 0) if explicit else None
        v.gups(0, log2_table, nupd, W.subseed(base, W.TAG_OPS), 3, acc=acc, launch=launch)
        assert int(acc.item()) == int(want)
        assert_no_device_errors()
