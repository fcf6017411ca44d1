"""The data-movement collectives where their work is cut differently: blocks
below and above a batch, a chunk and a round of work-groups, at bases and
sizes that are not multiples of 16, for teams that are no power of two."""
import numpy as np
import pytest

import oracle
import workload as W
from tests.gpu_helpers import assert_no_device_errors, download, heap, torch, upload

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


@pytest.mark.parametrize("npes", [9, 40, 70])   # one lane per vector; members over wavefronts; blocks of 64 in the edges
@pytest.mark.parametrize("dt", [oracle.DT_INT64, oracle.DT_FP32, oracle.DT_BF16])
def test_reductions_at_every_offset(dt, npes):
    """Sources and destinations at different offsets from a 16-byte boundary,
    and counts around the single elements at the edges and the shares of a
    work-group: bit-exact against the oracle, nothing else written."""
    es = {oracle.DT_INT64: 8, oracle.DT_FP32: 4, oracle.DT_BF16: 2}[dt]
    kmax = 33000
    with heap(npes, 1 << 20) as v:
        src, dst = v.malloc(kmax * es + 64), v.malloc(kmax * es + 64)
        so, do = v.offset(src), v.offset(dst)
        region = do + kmax * es + 64
        gen = {oracle.DT_INT64: W.coll_i64, oracle.DT_FP32: W.coll_f32, oracle.DT_BF16: W.coll_bf16}[dt]
        rows = np.stack([np.ascontiguousarray(gen(0xD0 + npes, p, kmax)).view(np.uint8) for p in range(npes)])
        for n in (1, 5, 16 // es, 31, 1000, kmax):
            for a, b in ((0, 0), (es, es), (0, es), (2 * es, 0), (16 - es, es)):
                for launch in (None, v.launch_cfg(wgs_per_pe=1, wg_size=64)):
                    init = W.heap_fill(0xD1, npes, region)
                    init[:, so + a:so + a + n * es] = rows[:, :n * es]
                    upload(init)
                    rop = oracle.RO_MAX if n == 31 else oracle.RO_SUM
                    v.reduce(dt, rop, dst + b, src + a, n, launch=launch)
                    ref = init.copy()
                    oracle.reduce(ref, dt, rop, do + b, so + a, n)
                    assert np.array_equal(download(region), ref), (n, a, b, launch is None)
        assert_no_device_errors()


@pytest.mark.parametrize("npes,eighths", [(23, 3), (24, 3), (33, 4), (56, 4), (57, 5), (64, 5)])
def test_reductions_split_over_wavefronts(npes, eighths):
    """Teams on both sides of those whose small reductions split the members
    over wavefronts, with the vectors of a launch around its limit: bit-exact
    against the oracle, in place as well."""
    with heap(npes, 2 << 20) as v:
        cus = torch().cuda.get_device_properties(0).multi_processor_count
        limit = eighths * cus * 32
        room = (limit + 1) * 16
        src, dst = v.malloc(room), v.malloc(room)
        so, do = v.offset(src), v.offset(dst)
        for dt, es, gen in ((oracle.DT_FP32, 4, W.coll_f32), (oracle.DT_BF16, 2, W.coll_bf16)):
            for nvec in (63, 65, limit, limit + 1):
                n = nvec * 16 // es
                init = W.heap_fill(0xD8, npes, do + room)
                for p in range(npes):
                    init[p, so:so + n * es] = np.ascontiguousarray(gen(0xD7, p, n)).view(np.uint8)
                for to, off in ((dst, do), (src, so)):
                    upload(init)
                    v.reduce(dt, oracle.RO_SUM, to, src, n)
                    ref = init.copy()
                    oracle.reduce(ref, dt, oracle.RO_SUM, off, so, n)
                    assert np.array_equal(download(do + room), ref), (dt, nvec, to == src)
        assert_no_device_errors()


@pytest.mark.parametrize("wgs,wg,chunk", [(1, 64, 4096), (7, 64, 0), (8, 64, 0), (1, 512, 8192), (1, 576, 32768)])
@pytest.mark.parametrize("kind", ["broadcast", "fcollect"])
def test_movement_with_few_wavefronts(kind, wgs, wg, chunk):
    """Launches on both sides of eight wavefronts per member, and small
    work-groups whose tasks are a few vectors per lane, for 17 members."""
    npes = 17
    with heap(npes, 4 << 20) as v:
        src, dst = v.malloc(200064), v.malloc(npes * 200064 + 64)
        so, do = v.offset(src), v.offset(dst)
        launch = v.launch_cfg(wgs_per_pe=wgs, wg_size=wg, chunk_bytes=chunk)
        for n in (7, 64, 4096, 16383, 16384, 32769, 200001):
            init = W.heap_fill(0xFE, npes, do + npes * 200064 + 64)
            for a, b in ((0, 0), (3, 5)):
                upload(init)
                ref = init.copy()
                if kind == "broadcast":
                    v.broadcastmem(dst + b, src + a, n, 3, launch=launch)
                    ref[:, do + b:do + b + n] = init[3, so + a:so + a + n]
                else:
                    v.fcollectmem(dst + b, src + a, n, launch=launch)
                    for q in range(npes):
                        ref[:, do + b + q * n:do + b + (q + 1) * n] = init[q, so + a:so + a + n]
                assert np.array_equal(download(init.shape[1]), ref), (n, a, b)
        assert_no_device_errors()
