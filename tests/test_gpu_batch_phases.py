"""Batches with more phases and tasks than a launch stages ahead, and many
atomics on few words in one phase, as plans and as device tables."""
import numpy as np
import pytest

import oracle
import workload as W
from tests.gpu_helpers import assert_no_device_errors, download, heap, torch, upload

pytestmark = pytest.mark.gpu


def _launchers(v, descs, results):
    t = torch()
    plan = v.Plan(descs)
    table = t.from_numpy(np.ascontiguousarray(descs).view(np.uint8).copy()).cuda()
    return {"plan": lambda: plan.launch_fused(results=results),
            "table": lambda: v.launch_batch(table, len(descs), results=results)}


@pytest.mark.parametrize("wg_size,grid_wgs", [(64, 0), (256, 3), (1024, 0)])
def test_many_phases_and_tasks(wg_size, grid_wgs):
    """40 epochs of mixed scopes (a grid of three work-groups has several
    tasks per phase), launched three times over with eager work between."""
    npes = 3
    wl = W.small_workload(seed=0x9A5E, npes=npes, heap_bytes=1 << 18, n_rma=1600, epoch_ops=40, n_amo=200)
    d = wl.descs.copy()
    rma = np.isin(d["op"], (W.OP_PUT, W.OP_GET))
    d["scope"][rma] = np.arange(int(rma.sum())) % 3
    with heap(npes, 1 << 18) as v:
        tune = v.default_tune()
        tune.wg_size, tune.grid_wgs = wg_size, grid_wgs
        t = torch()
        plan = v.Plan(d, tune)
        assert plan.info()["phases"] > 16
        res = t.zeros(wl.n_amo, dtype=t.int64, device="cuda")
        ref = wl.init.copy()
        upload(wl.init)
        side = t.zeros(1 << 20, device="cuda")
        for _ in range(3):
            plan.launch_fused(results=res)
            side += 1
            oracle.run_program(ref, d, nresults=wl.n_amo)
            assert np.array_equal(download(wl.heap_bytes), ref)
        assert_no_device_errors()


@pytest.mark.parametrize("nwords", [1, 3, 64, 700])
@pytest.mark.parametrize("form", ["plan", "table"])
def test_contended_adds_and_xors(form, nwords):
    """fetch_add, add, fetch_xor and xor of arbitrary values on few words in
    one phase, other atomics and short puts among them: the final words are
    the closed forms, and each word's fetched values are one serial order."""
    npes, nops = 2, 3000
    x = W.splitmix64(0xADD, 0, 3 * nops)
    with heap(npes, 1 << 20) as v:
        t = torch()
        init = W.heap_fill(0xADD1, npes, 16384 + 8 * nops + 8)
        recs, words = [], {}
        for i in range(nops):
            w = int(x[3 * i] % np.uint64(nwords))
            xor = w % 2 == 1
            fetch = w % 5 != 2      # words 2, 7, ... take the forms that fetch nothing
            val = int(x[3 * i + 1]) if xor else 1 + int(x[3 * i + 1] % np.uint64(1 << 40))
            op = ((W.OP_AMO_FETCH_XOR if fetch else W.OP_AMO_XOR) if xor
                  else (W.OP_AMO_FETCH_ADD if fetch else W.OP_AMO_ADD))
            pe = w % npes
            recs.append((op, W.SCOPE_THREAD, 0, i % npes, pe, i if fetch else W.NO_RESULT, 8 * w, 0, 8, val, 0))
            words.setdefault((pe, w, xor), []).append((i if fetch else None, val))
            if i % 97 == 0:   # others in the same packs, on words and bytes of their own
                recs.append((W.OP_AMO_SET, W.SCOPE_THREAD, 0, 0, 1, W.NO_RESULT, 16384 + 8 * i, 0, 8, i, 0))
        d = W.descs(recs)
        ref = init.copy()
        for (pe, w, xor), ops in words.items():
            cell = ref[pe, 8 * w:8 * w + 8].view(np.uint64)
            for _, val in ops:
                with np.errstate(over="ignore"):
                    cell[0] = cell[0] ^ np.uint64(val) if xor else cell[0] + np.uint64(val)
        for i in range(0, nops, 97):
            ref[1, 16384 + 8 * i:16384 + 8 * i + 8].view(np.uint64)[0] = i
        upload(init)
        res = t.zeros(len(d), dtype=t.int64, device="cuda")
        _launchers(v, d, res)[form]()
        assert np.array_equal(download(init.shape[1]), ref)
        got = res.cpu().numpy().view(np.uint64)
        M = (1 << 64) - 1
        for (pe, w, xor), ops in words.items():
            if ops[0][0] is None:
                continue   # nothing fetched: the closed form above
            nxt = {int(got[i]): val for i, val in ops}
            assert len(nxt) == len(ops)
            cur = int(init[pe, 8 * w:8 * w + 8].view(np.uint64)[0])
            for _ in ops:
                cur = (cur ^ nxt[cur]) if xor else (cur + nxt[cur]) & M
            assert cur == int(ref[pe, 8 * w:8 * w + 8].view(np.uint64)[0])
        assert_no_device_errors()


@pytest.mark.parametrize("case", ["one_tile", "tile_edge", "points_at_limit", "points_past_limit", "large_table",
                                  "many_tasks", "unequal_barriers"])
def test_index_forms(case):
    """Tables on both sides of what the parallel index takes: whole tiles of
    1024 descriptors and one more, 1024 ordering points and more, more than
    65536 descriptors, an operation of 65536 work-group tasks; and a table
    whose PEs see different numbers of barriers, of which nothing runs."""
    npes, size = 3, 1 << 21
    x = W.splitmix64(0x1DE, 0, 4096)
    recs, ref_ops = [], []

    def sync(op, pe):
        recs.append((op, W.SCOPE_WG, 0, pe, pe, W.NO_RESULT, 0, 0, 0, 0, 0))

    def put(k, n=24, scope=W.SCOPE_AUTO):   # slot k of the target's second half, from the issuer's first
        pe = k % npes
        recs.append((W.OP_PUT, scope, 0, pe, (pe + 1) % npes, W.NO_RESULT, 64 * (k % 8192), size // 2 + 64 * (k % 8192),
                     n, 0, 0))

    def epoch(count, at=0, fences=0):
        for k in range(count):
            put(at + k, 8 + int(x[k % 4096] % np.uint64(56)), (W.SCOPE_AUTO, W.SCOPE_WAVE, W.SCOPE_WG)[k % 3])
            if fences and k % max(1, count // fences) == 0:
                sync(W.OP_FENCE, k % npes)
        for p in range(npes):
            sync(W.OP_BARRIER_ALL, p)

    if case == "one_tile":
        epoch(1021)
    elif case == "tile_edge":
        epoch(500, fences=7), epoch(520), epoch(1500, fences=3)
        assert len(recs) > 2048
    elif case in ("points_at_limit", "points_past_limit"):
        for e in range(341):
            epoch(3, at=3 * e)
        sync(W.OP_FENCE, 0)
        if case == "points_past_limit":
            sync(W.OP_QUIET, 1)
        put(7777)
    elif case == "large_table":
        for e in range(9):
            epoch(8000)
        assert len(recs) > 65536
    elif case == "many_tasks":
        epoch(40)
        recs.append((W.OP_PUT, W.SCOPE_WG, 0, 0, 1, W.NO_RESULT, 0, size // 2, size // 2, 0, 0))
    else:
        epoch(100)
        sync(W.OP_BARRIER_ALL, 1)
        put(5)
    d = W.descs(recs)
    with heap(npes, size) as v:
        t = torch()
        init = W.heap_fill(0x1DE, npes, size)
        upload(init)
        table = t.from_numpy(np.ascontiguousarray(d).view(np.uint8).copy()).cuda()
        tune = v.default_tune()
        if case == "many_tasks":
            for c in range(len(tune.chunk)):
                tune.chunk[c] = 16
        dt = t.frombuffer(bytearray(bytes(tune)), dtype=t.uint8).cuda()
        ref = init.copy()
        if case != "unequal_barriers":
            oracle.run_program(ref, d)
        for _ in range(2):
            v.launch_batch(table, len(d), d_tune=dt)
            assert np.array_equal(download(size), ref)
        want = v.DEVERR_BAD_DESC if case == "unequal_barriers" else 0
        assert v.device_errors() == want
