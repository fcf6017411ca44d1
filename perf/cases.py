"""Performance cases of the framework: what is timed, on which inputs, and
what a pass returns.

A case is one call that a program makes on a symmetric heap it has set up:
a round of put/get messages, a team collective, a reduction, a round of
atomics, or a mixed program (a host-built plan, or a descriptor table in
device memory).  prepare() gives what the program holds before the call: the
library initialised for the case's PEs, symmetric objects with their inputs,
launch shapes, plans and tables.  run() is the call.  Inputs come from torch's
own generator, so that exact() needs none of the framework's code.

Serving (the persistent progress kernel) is not a case: where a request's
result lands depends on the arrival times of a run.
"""
import math

import torch

MIB = 1 << 20
KINDS = ("put", "get", "alltoall", "fcollect", "broadcast", "reduce", "gups", "plan", "table")


# ---------------------------------------------------------------- the cases
def _rma(name, op, scope, npes, size, nmsg, pattern, src_shift=0, dst_shift=0, gap=0):
    return {"name": name, "kind": op, "scope": scope, "npes": npes, "size": size, "nmsg": nmsg, "pattern": pattern,
            "src_shift": src_shift, "dst_shift": dst_shift, "gap": gap}


def _coll(name, kind, npes, size, start=0, stride=1, members=0, shift=0):
    return {"name": name, "kind": kind, "npes": npes, "size": size, "start": start, "stride": stride,
            "members": members or npes, "shift": shift}


def _red(name, dtype, op, npes, count, start=0, stride=1, members=0, shift=0):
    return {"name": name, "kind": "reduce", "dtype": dtype, "op": op, "npes": npes, "count": count, "start": start,
            "stride": stride, "members": members or npes, "shift": shift}


def _prog(name, kind, npes, n_rma, epoch, n_amo, max_size):
    return {"name": name, "kind": kind, "npes": npes, "n_rma": n_rma, "epoch": epoch, "n_amo": n_amo,
            "max_size": max_size}


def listed():
    return [
        # The largest moves: every PE streams 16 MiB messages to its neighbour.
        _rma("put_wg_16MiB_ring", "put", "wg", 64, 16 * MIB, 4, "ring"),
        # Ordinary messages, one wavefront each (halo rows, key/value pages).
        _rma("get_wave_1KiB_perm", "get", "wave", 64, 1024, 8192, "perm"),
        # Fine-grained messages, one lane each.
        _rma("put_thread_64B_ring", "put", "thread", 64, 64, 16384, "ring"),
        # Packed records of odd length at odd addresses (a ragged exchange).
        _rma("get_wave_ragged_1501B", "get", "wave", 64, 1501, 4096, "perm", src_shift=3, dst_shift=8),
        # The small exchange of every step, where latency counts.
        _coll("alltoall_4KiB", "alltoall", 64, 4096),
        # A gather of ragged rows: a block size that is no multiple of a vector.
        _coll("fcollect_100001B", "fcollect", 64, 100001),
        # A parameter block from one PE to all.
        _coll("broadcast_1MiB", "broadcast", 64, MIB),
        # One gradient bucket.
        _red("reduce_f32_sum_256Ki", "f32", "sum", 64, 1 << 18),
        # A large bf16 vector of odd length.
        _red("reduce_bf16_sum_4000003", "bf16", "sum", 64, 4000003),
        # Random-access atomics on a table spread over the PEs.
        {"name": "gups_16M_updates", "kind": "gups", "npes": 64, "log2_table": 27, "updates": 1 << 24},
        # The small mixed program (put/get epochs, then contended fetch_add),
        # as a plan that the program built once ...
        _prog("program_plan_4pe", "plan", 4, 1000, 125, 10000, 4096),
        # ... and as a table in device memory, which a kernel may have written.
        _prog("program_table_4pe", "table", 4, 1000, 125, 10000, 4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _team(rng, npes):
    """(start, stride, members) of a team: mostly everyone, sometimes a strided part."""
    if npes < 4 or rng.random() < 0.7:
        return 0, 1, npes
    stride = rng.choice((1, 2))
    start = rng.randrange(0, npes // 4 + 1)
    return start, stride, rng.randrange(2, (npes - 1 - start) // stride + 2)


def draw(rng):
    case = _draw(rng)
    case.pop("name", None)
    return case


def _draw(rng):
    kind = rng.choice(KINDS)
    if kind in ("put", "get"):
        scope = rng.choice(("thread", "wave", "wg", "grid"))
        npes = rng.choice((rng.randrange(2, 65), 64))
        hi = {"thread": 2048, "wave": MIB, "wg": 16 * MIB, "grid": 16 * MIB}[scope]
        lo = {"thread": 8, "wave": 64, "wg": 1024, "grid": 65536}[scope]
        size = _log_int(rng, lo, hi)
        ragged = rng.random() < 0.5
        if not ragged:
            size = max(8, size // 16 * 16 if size >= 16 else 8)
        cap = {"thread": 16384, "wave": 4096, "wg": 1024, "grid": 16}[scope]
        nmsg = max(1, min(cap, 32 * MIB // size))
        return _rma("", kind, scope, npes, size, nmsg, rng.choice(("ring", "perm")),
                    rng.randrange(16) if ragged else 0, rng.randrange(16) if ragged else 0,
                    rng.choice((0, rng.randrange(1, 64))) if ragged else 0)
    if kind in ("alltoall", "fcollect", "broadcast"):
        npes = rng.choice((rng.randrange(2, 65), 64))
        start, stride, members = _team(rng, npes)
        hi = {"alltoall": MIB, "fcollect": MIB, "broadcast": 32 * MIB}[kind] // (4 if members > 32 else 1)
        size = _log_int(rng, 16, hi)
        ragged = rng.random() < 0.4
        if not ragged:
            size = size // 16 * 16
        return _coll("", kind, npes, size, start, stride, members, rng.randrange(16) if ragged else 0)
    if kind == "reduce":
        npes = rng.choice((rng.randrange(2, 65), 64))
        start, stride, members = _team(rng, npes)
        count = _log_int(rng, 16, 1 << 21)
        ragged = rng.random() < 0.5
        if not ragged:
            count = count // 8 * 8
        return _red("", rng.choice(("i64", "f32", "bf16")), rng.choice(("sum", "max")), npes, count, start, stride,
                    members, rng.randrange(4) if ragged else 0)
    if kind == "gups":
        return {"kind": "gups", "npes": rng.choice((4, 16, 64)), "log2_table": rng.randrange(18, 28),
                "updates": _log_int(rng, 1 << 14, 1 << 24)}
    npes = rng.randrange(2, 17)
    return _prog("", kind, npes, rng.randrange(100, 1500), rng.randrange(40, 200), rng.randrange(0, 12000),
                 _log_int(rng, 256, 16384))


# ------------------------------------------------------------------- inputs
def _gen(seed, tag):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1000003 + tag) & 0x7FFFFFFFFFFFFFFF)


def _bytes(seed, tag, rows, n):
    """(rows, n) random bytes."""
    g = _gen(seed, tag)
    w = torch.randint(-(1 << 63), (1 << 63) - 1, (rows, (n + 7) // 8), dtype=torch.int64, device="cuda", generator=g)
    return w.view(torch.uint8)[:, :n]


_TYPES = {"i64": (torch.int64, 8), "f32": (torch.float32, 4), "bf16": (torch.bfloat16, 2)}


def _elements(seed, dtype, rows, n):
    """(rows, n) elements: raw int64 words, or floats uniform over [-1, 1)."""
    g = _gen(seed, 1)
    if dtype == "i64":
        return torch.randint(-(1 << 63), (1 << 63) - 1, (rows, n), dtype=torch.int64, device="cuda", generator=g)
    x = torch.rand((rows, n), dtype=torch.float32, device="cuda", generator=g) * 2 - 1
    return x.to(_TYPES[dtype][0])


# ------------------------------------------------------------------ session
class _Session:
    """The library as a program initialises it: one heap for its PEs."""

    npes = 0
    user = 0
    epoch = 0
    teams = {}


def _heap(npes, per_state):
    """Initialise the library for `npes` PEs with room for four states."""
    import paper_2607_08006_amd as v

    need = max(4 * per_state + 4 * MIB, (1 << 30) if npes == 64 else 64 * MIB)
    if _Session.npes != npes or _Session.user < need or not v.initialized():
        if v.initialized():
            torch.cuda.synchronize()
            v.finalize()
            torch.cuda.empty_cache()
        v.init(npes, need)
        _Session.npes, _Session.user = npes, need
        _Session.epoch += 1
        _Session.teams = {}
    return v


class _State:
    """A program's symmetric objects and call; the objects go back to the
    heap with it."""

    def __init__(self, v):
        self.v, self.epoch, self.objects, self.keep = v, _Session.epoch, [], []
        self.call = self.out = None

    def alloc(self, n):
        p = self.v.align(4096, n)
        self.objects.append(p)
        return self.v.offset(p)

    def __del__(self):
        try:
            if self.epoch == _Session.epoch and self.v.initialized():
                torch.cuda.synchronize()
                for p in self.objects:
                    self.v.free(p)
        except Exception:
            pass


def _team_of(v, case):
    """(team handle, its PEs)."""
    start, stride, members = case["start"], case["stride"], case["members"]
    pes = range(start, start + stride * members, stride)
    if start == 0 and stride == 1 and members == case["npes"]:
        return v.DEVICE_TEAM_WORLD, pes
    key = (start, stride, members)
    if key not in _Session.teams:
        _Session.teams[key] = v.team_split_strided(v.TEAM_WORLD, start, stride, members)
    return _Session.teams[key], pes


def _rows(v, pes, off, n):
    """Bytes [off, off + n) of the given PEs' slices, as a view of the heap."""
    rows = v.heap_view()[pes.start:pes.stop:pes.step, off:off + n]
    # Whole words where the range allows it: the same bytes, fewer elements.
    return rows.view(torch.int64) if off % 8 == 0 and n % 8 == 0 else rows


def _launch(v, scope, size):
    """The launch shapes of the benchmark's bandwidth sweep."""
    nt, deep = v.LAUNCH_NONTEMPORAL, v.LAUNCH_DEEP
    if scope == "thread":
        return v.launch_cfg(wgs_per_pe=2, wg_size=1024) if size <= 32 else v.launch_cfg(wgs_per_pe=4, wg_size=256)
    if scope == "wave":
        return v.launch_cfg(wgs_per_pe=4, wg_size=256, flags=nt if size >= 4096 else 0)
    if scope == "wg":
        return v.launch_cfg(wgs_per_pe=4, wg_size=1024, flags=(nt | deep) if size >= 65536 else 0)
    return v.launch_cfg(wgs_per_pe=4, wg_size=256, flags=nt | deep)


def _prepare_rma(case, seed):
    import workload as W

    npes, size, k = case["npes"], case["size"], case["nmsg"]
    step = size + case["gap"]
    span = k * step + 64
    v = _heap(npes, 2 * span + 3 * 4096)
    s = _State(v)
    src, dst = s.alloc(span), s.alloc(span)
    h = v.heap_view()
    h[:, src:src + span].copy_(_bytes(seed, 0, npes, span))
    h[:, dst:dst + span].zero_()
    targets = W.ring(npes) if case["pattern"] == "ring" else W.derangement(seed, npes)
    tg = torch.from_numpy(targets.astype("int32")).cuda()
    op = v.OP_PUT if case["kind"] == "put" else v.OP_GET
    scope = {"thread": v.SCOPE_THREAD, "wave": v.SCOPE_WAVE, "wg": v.SCOPE_WG, "grid": v.SCOPE_GRID}[case["scope"]]
    lc = _launch(v, case["scope"], size)
    a, b = src + case["src_shift"], dst + case["dst_shift"]
    s.call = lambda: v.rma_pattern(op, scope, tg, a, b, size, k, src_step=step, dst_step=step, launch=lc)
    s.out = _rows(v, range(npes), dst, (span + 7) // 8 * 8)
    return s


def _prepare_coll(case, seed):
    kind, npes, n, P = case["kind"], case["npes"], case["size"], case["members"]
    sn = n * P if kind == "alltoall" else n
    dn = n if kind == "broadcast" else n * P
    v = _heap(npes, sn + dn + 128 + 3 * 4096)
    s = _State(v)
    src, dst = s.alloc(sn + 64), s.alloc(dn + 64)
    team, pes = _team_of(v, case)
    h = v.heap_view()
    h[:, src:src + sn + 64].copy_(_bytes(seed, 0, npes, sn + 64))
    h[:, dst:dst + dn + 64].zero_()
    base = v.heap_base()
    a, b = base + src, base + dst + case["shift"]
    if kind == "broadcast":
        root = seed % P
        s.call = lambda: v.broadcastmem(b, a, n, root, team=team)
    elif kind == "fcollect":
        s.call = lambda: v.fcollectmem(b, a, n, team=team)
    else:
        s.call = lambda: v.alltoallmem(b, a, n, team=team)
    s.out = _rows(v, pes, dst, (dn + case["shift"] + 7) // 8 * 8)
    return s


def _prepare_reduce(case, seed):
    npes, n, P = case["npes"], case["count"], case["members"]
    dtype, es = _TYPES[case["dtype"]]
    shift = case["shift"] * es
    v = _heap(npes, 2 * n * es + 128 + 3 * 4096)
    s = _State(v)
    src, dst = s.alloc(n * es), s.alloc(n * es + 64)
    team, pes = _team_of(v, case)
    h = v.heap_view()
    h[pes.start:pes.stop:pes.step, src:src + n * es].view(dtype).copy_(_elements(seed, case["dtype"], P, n))
    base = v.heap_base()
    dt = {"i64": v.DT_INT64, "f32": v.DT_FP32, "bf16": v.DT_BF16}[case["dtype"]]
    op = v.RED_SUM if case["op"] == "sum" else v.RED_MAX
    s.call = lambda: v.reduce(dt, op, base + dst + shift, base + src, n, team=team)
    s.out = h[pes.start:pes.stop:pes.step, dst + shift:dst + shift + n * es].view(dtype)
    return s


def _prepare_gups(case, seed):
    npes, lt = case["npes"], case["log2_table"]
    n = 8 << (lt - int(math.log2(npes)))
    v = _heap(npes, n + 2 * 4096)
    s = _State(v)
    tab = s.alloc(n)
    v.heap_view()[:, tab:tab + n].copy_(_bytes(seed, 0, npes, n))
    acc = torch.zeros(1, dtype=torch.int64, device="cuda")
    # Adds only: the table after a pass is one whatever the order of updates.
    s.call = lambda: v.gups(tab, lt, case["updates"], seed, 1, acc=acc)
    s.out = _rows(v, range(npes), tab, n)
    return s


def _prepare_program(case, seed):
    import numpy as np
    import workload as W

    npes = case["npes"]
    per_pe = -(-(case["epoch"] * case["max_size"] * 2) // npes) + 65536
    size = max(MIB, 1 << (per_pe - 1).bit_length())
    v = _heap(npes, size + 2 * 4096)
    s = _State(v)
    off = s.alloc(size)
    wl = W.small_workload(seed, npes=npes, heap_bytes=size, n_rma=case["n_rma"], epoch_ops=case["epoch"],
                          n_amo=case["n_amo"], max_size=case["max_size"], base_off=off, fill=False)
    h = v.heap_view()
    h[:, off:off + size].copy_(_bytes(seed, 0, npes, size))
    h[:, off + wl.counter_off:off + wl.counter_off + 8 * wl.ncounters].zero_()
    nd = len(wl.descs)
    res = torch.zeros(nd, dtype=torch.int64, device="cuda")
    if case["kind"] == "plan":
        plan = v.Plan(wl.descs)
        s.call = lambda: plan.launch_fused(results=res)
    else:
        table = torch.from_numpy(np.ascontiguousarray(wl.descs).view(np.uint8).copy()).cuda()
        s.call = lambda: v.launch_batch(table, nd, results=res)
    # The fetched values are any serial order of the contended counters; the
    # heap they leave is one.
    s.out = _rows(v, range(npes), off, size)
    return s


_PREPARE = {"put": _prepare_rma, "get": _prepare_rma, "alltoall": _prepare_coll, "fcollect": _prepare_coll,
            "broadcast": _prepare_coll, "reduce": _prepare_reduce, "gups": _prepare_gups, "plan": _prepare_program,
            "table": _prepare_program}


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


def run(state):
    state.call()
    return state.out


# --------------------------------------------------------------------- work
def work(case):
    """Bytes the definition of the pass reads and writes, each once, and the
    reductions' additions or comparisons."""
    kind = case["kind"]
    if kind in ("put", "get"):
        return {"bytes": 2 * case["npes"] * case["nmsg"] * case["size"], "flops": 0}
    if kind == "alltoall":
        return {"bytes": 2 * case["members"] ** 2 * case["size"], "flops": 0}
    if kind == "fcollect":
        return {"bytes": (case["members"] + case["members"] ** 2) * case["size"], "flops": 0}
    if kind == "broadcast":
        return {"bytes": (1 + case["members"]) * case["size"], "flops": 0}
    if kind == "reduce":
        es = _TYPES[case["dtype"]][1]
        return {"bytes": 2 * case["members"] * case["count"] * es, "flops": (case["members"] - 1) * case["count"]}
    if kind == "gups":
        return {"bytes": 16 * case["updates"], "flops": 0}
    ops = case["n_rma"] + case["n_amo"]
    payload = case["n_rma"] * (8 + case["max_size"]) // 2
    return {"bytes": 2 * payload + 16 * case["n_amo"] + 64 * ops, "flops": 0}


# -------------------------------------------------------------------- exact
def exact(case, seed):
    """The reductions in 64 bits; what is moved or counted has no rounding."""
    if case["kind"] != "reduce":
        return None
    x = _elements(seed, case["dtype"], case["members"], case["count"])
    if case["dtype"] != "i64":
        x = x.double()
    r = x.sum(0) if case["op"] == "sum" else x.max(0).values
    return r.expand(case["members"], case["count"])
