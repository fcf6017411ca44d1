"""The data-movement collectives where their work is cut differently: blocks
below and above a batch, a chunk and a round of work-groups, at bases and
sizes that are not multiples of 16, for teams that are no power of two."""
import numpy as np
import pytest

import workload as W
from tests.gpu_helpers import assert_no_device_errors, download, heap, upload

pytestmark = pytest.mark.gpu

SIZES = [1, 15, 16, 129, 8208, 16383, 16384, 65537, 300001]
BIG = [3000001]


@pytest.mark.parametrize("launch", [None, dict(wgs_per_pe=3, wg_size=192, chunk_bytes=4112)])
@pytest.mark.parametrize("npes,team", [(13, None), (13, (2, 3, 4))])
@pytest.mark.parametrize("kind", ["broadcast", "fcollect", "alltoall"])
def test_movement_at_split_edges(kind, npes, team, launch):
    room = npes * 300001 + 4096
    with heap(npes, 2 * room + (1 << 20)) as v:
        handle, pes = v.DEVICE_TEAM_WORLD, list(range(npes))
        if team:
            handle = v.team_split_strided(v.TEAM_WORLD, *team)
            pes = [team[0] + k * team[1] for k in range(team[2])]
        P = len(pes)
        src, dst = v.malloc(room), v.malloc(room + 64)
        so, do = v.offset(src), v.offset(dst)
        init = W.heap_fill(0xC0 + npes, npes, do + room + 64)
        L = v.launch_cfg(**launch) if launch else None
        for n in SIZES + (BIG if kind == "broadcast" and not launch else []):
            if n * (1 if kind == "broadcast" else P) + 32 > room:
                continue
            for ss, ds in ((0, 0), (5, 3)):
                upload(init)
                ref = init.copy()
                a, b = so + ss, do + ds
                if kind == "broadcast":
                    v.broadcastmem(dst + ds, src + ss, n, P - 1, team=handle, launch=L)
                    for p in pes:
                        ref[p, b:b + n] = init[pes[P - 1], a:a + n]
                elif kind == "fcollect":
                    v.fcollectmem(dst + ds, src + ss, n, team=handle, launch=L)
                    for p in pes:
                        for q in range(P):
                            ref[p, b + q * n:b + (q + 1) * n] = init[pes[q], a:a + n]
                else:
                    v.alltoallmem(dst + ds, src + ss, n, team=handle, launch=L)
                    for k, p in enumerate(pes):
                        for q in range(P):
                            ref[p, b + q * n:b + (q + 1) * n] = init[pes[q], a + k * n:a + (k + 1) * n]
                assert np.array_equal(download(init.shape[1]), ref), (n, ss, ds)
        assert_no_device_errors()
