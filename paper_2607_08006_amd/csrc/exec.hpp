// Executors of single descriptor operations, shared by the batched forms
// (plans built on the host, descriptor tables in device memory) and their
// per-operation launches.  Internal to the library.
#pragma once
#include "runtime.hpp"

namespace vshmem_exec {

// Host and device: whether an op code is a fence, quiet or barrier, and
// whether it is an atomic.
__host__ __device__ __forceinline__ bool is_sync_op(uint8_t op)
{
    return op == SHMEMX_OP_FENCE || op == SHMEMX_OP_QUIET || op == SHMEMX_OP_BARRIER_ALL;
}
__host__ __device__ __forceinline__ bool is_amo_op(uint8_t op)
{
    return op >= SHMEMX_OP_AMO_FETCH_ADD && op <= SHMEMX_OP_AMO_SWAP;
}
// Size class of a message: floor(log2(n)), capped at the table's last class.
__host__ __device__ __forceinline__ int size_class(uint64_t n)
{
    int c = 0;
    while (c + 1 < SHMEMX_TUNE_CLASSES && (2ull << c) <= n) ++c;
    return c;
}
// Scope an operation executes at: an explicit scope, else the table's
// choice for its size class (atomics: one lane).
__host__ __device__ __forceinline__ int resolve_scope(const shmemx_desc_t &d, const shmemx_tune_t &tune)
{
    if (is_amo_op(d.op)) return d.scope == SHMEMX_SCOPE_AUTO ? SHMEMX_SCOPE_THREAD : d.scope;
    if (d.scope != SHMEMX_SCOPE_AUTO) return d.scope;
    return tune.scope[size_class(d.nbytes)];
}
// Bytes per work-group task of an operation at `scope`: the table's chunk
// for its class (grid scope: 256 KiB when the table has none), rounded up
// to 16; signal-puts and atomics are never split.
__host__ __device__ __forceinline__ uint64_t resolve_chunk(const shmemx_desc_t &d, int scope, const shmemx_tune_t &tune)
{
    if (d.op == SHMEMX_OP_PUT_SIGNAL || is_amo_op(d.op)) return d.nbytes ? d.nbytes : 1;
    uint64_t ch = tune.chunk[size_class(d.nbytes)];
    if (scope == SHMEMX_SCOPE_GRID && ch == 0) ch = 256ull << 10;
    if (ch == 0 || ch >= d.nbytes) return d.nbytes ? d.nbytes : 1;
    return (ch + 15) & ~15ull;
}

__device__ __forceinline__ uint64_t *amo_word(const shmemx_dctx_pub_t &c, const shmemx_desc_t &d)
{
    return (uint64_t *)(c.base + (uint64_t)d.target_pe * c.stride + d.src);
}

// Atomics and signal-free single-lane work.
__device__ __forceinline__ void exec_amo(const shmemx_dctx_pub_t &c, const shmemx_desc_t &d, uint64_t *results)
{
    uint64_t *w = amo_word(c, d);
    uint64_t old = 0;
    bool fetch = true;
    switch (d.op) {
    case SHMEMX_OP_AMO_FETCH_ADD: old = __hip_atomic_fetch_add(w, d.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); break;
    case SHMEMX_OP_AMO_FETCH_XOR: old = __hip_atomic_fetch_xor(w, d.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); break;
    case SHMEMX_OP_AMO_COMPARE_SWAP: {
        uint64_t e = d.cond;
        __hip_atomic_compare_exchange_strong(w, &e, d.value, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        old = e;
        break;
    }
    case SHMEMX_OP_AMO_ADD:
        __hip_atomic_fetch_add(w, d.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        fetch = false;
        break;
    case SHMEMX_OP_AMO_XOR:
        __hip_atomic_fetch_xor(w, d.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        fetch = false;
        break;
    case SHMEMX_OP_AMO_SET:
        __hip_atomic_store(w, d.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        fetch = false;
        break;
    case SHMEMX_OP_AMO_FETCH: old = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); break;
    case SHMEMX_OP_AMO_SWAP: old = __hip_atomic_exchange(w, d.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); break;
    default: fetch = false;
    }
    if (fetch && results && d.result_idx != SHMEMX_NO_RESULT) results[d.result_idx] = old;
}

// Byte range [lo, hi) of a put/get, copied by nl lanes (LONE: by one lane).
// SHORT (copy_bytes) pays for work-groups only: the mixed program of 4 PEs
// all at work-group scope 43.5 us without and 40.1 with.
template <bool LONE = false, bool SHORT = false>
__device__ __forceinline__ void exec_copy(const shmemx_dctx_pub_t &c, const shmemx_desc_t &d, uint64_t lo, uint64_t hi,
                                          uint64_t lane, uint64_t nl)
{
    const bool get = d.op == SHMEMX_OP_GET;
    const int spe = get ? d.target_pe : d.issuer_pe;
    const int dpe = get ? d.issuer_pe : d.target_pe;
    const uint8_t *S = c.base + (uint64_t)spe * c.stride + d.src + lo;
    uint8_t *D = c.base + (uint64_t)dpe * c.stride + d.dst + lo;
    vshmem_detail::copy_bytes<VSHMEM_COPY_UNROLL, false, LONE, VSHMEM_COPY_UNROLL, SHORT>(D, S, hi - lo, lane, nl);
}

__device__ __forceinline__ void signal_of(const shmemx_dctx_pub_t &c, const shmemx_desc_t &d)
{
    uint64_t *s = (uint64_t *)(c.base + (uint64_t)d.target_pe * c.stride + d.cond);
    if (d.aux == SHMEM_SIGNAL_ADD)
        __hip_atomic_fetch_add(s, d.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        __hip_atomic_store(s, d.value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One operation by a single lane.
__device__ __forceinline__ void exec_thread(const shmemx_dctx_pub_t &c, const shmemx_desc_t &d, uint64_t *results)
{
    if (is_amo_op(d.op)) {
        exec_amo(c, d, results);
    } else if (d.op == SHMEMX_OP_PUT || d.op == SHMEMX_OP_GET || d.op == SHMEMX_OP_PUT_SIGNAL) {
        exec_copy<true>(c, d, 0, d.nbytes, 0, 1);
        if (d.op == SHMEMX_OP_PUT_SIGNAL) {
            vshmem_detail::release_agent();
            signal_of(c, d);
        }
    }
}

// One operation per lane, the wavefront's lanes 0 .. n - 1 calling together.
// Neighbouring lanes that add to (or xor) one word combine: one of them takes
// the word with the run's sum, the others derive the values that the word
// would have shown them, had they gone in lane order.  Atomics on one word
// serialise in memory (50 to 70 ns each on MI355X, in or out of one
// wavefront): 10^4 fetch_add on 64 counters took 7.3 us in program order and
// 11.7 sorted by word, and take 3.0 sorted and combined.
__device__ __forceinline__ void exec_lanes(const shmemx_dctx_pub_t &c, const shmemx_desc_t &d, uint64_t *results)
{
    const uint32_t lane = __lane_id();
    const bool add = d.op == SHMEMX_OP_AMO_FETCH_ADD || d.op == SHMEMX_OP_AMO_ADD;
    const bool combines = add || d.op == SHMEMX_OP_AMO_FETCH_XOR || d.op == SHMEMX_OP_AMO_XOR;
    // Words are 8-byte aligned: bit 0 tells xor from add, bit 2 a lane alone.
    uint64_t *w = amo_word(c, d);
    const uint64_t key = combines ? (uint64_t)w | (add ? 0 : 1) : ((uint64_t)lane << 3) | 4;
    const bool head = lane == 0 || __shfl_up(key, 1, 64) != key;
    const uint64_t heads = __ballot(head), active = __ballot(true);
    if (heads == active) {
        exec_thread(c, d, results);
        return;
    }
    // Inclusive scan over each run of equal keys.
    uint64_t x = combines ? d.value : 0;
    const uint32_t begin = 63 - (uint32_t)__builtin_clzll(heads & (~0ull >> (63 - lane)));
#pragma unroll
    for (uint32_t o = 1; o < 64; o <<= 1) {
        const uint64_t y = __shfl_up(x, o, 64);
        if (lane >= begin + o) x = add ? x + y : x ^ y;
    }
    const uint64_t later = lane == 63 ? 0 : heads >> (lane + 1) << (lane + 1);
    const uint32_t end = (later ? (uint32_t)__builtin_ctzll(later) : (uint32_t)__builtin_popcountll(active)) - 1;
    uint64_t old = 0;
    if (combines) {
        if (lane == end)
            old = add ? __hip_atomic_fetch_add(w, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                      : __hip_atomic_fetch_xor(w, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
        exec_thread(c, d, results);
    }
    old = __shfl(old, (int)end, 64);
    if (combines) {
        old = add ? old + (x - d.value) : old ^ x ^ d.value;
        const bool fetch = d.op == SHMEMX_OP_AMO_FETCH_ADD || d.op == SHMEMX_OP_AMO_FETCH_XOR;
        if (fetch && results && d.result_idx != SHMEMX_NO_RESULT) results[d.result_idx] = old;
    }
}

// One operation by a whole wavefront.
__device__ __forceinline__ void exec_wave(const shmemx_dctx_pub_t &c, const shmemx_desc_t &d, uint64_t *results)
{
    if (is_amo_op(d.op)) {
        if (__lane_id() == 0) exec_amo(c, d, results);
    } else if (d.op == SHMEMX_OP_PUT || d.op == SHMEMX_OP_GET || d.op == SHMEMX_OP_PUT_SIGNAL) {
        exec_copy(c, d, 0, d.nbytes, __lane_id(), 64);
        if (d.op == SHMEMX_OP_PUT_SIGNAL) {
            vshmem_detail::release_agent();
            if (__lane_id() == 0) signal_of(c, d);
        }
    }
}

// A byte range of one operation by a whole work-group.
__device__ __forceinline__ void exec_wg(const shmemx_dctx_pub_t &c, const shmemx_desc_t &d, uint64_t lo, uint64_t hi,
                                        uint64_t *results)
{
    if (is_amo_op(d.op)) {
        if (threadIdx.x == 0) exec_amo(c, d, results);
    } else if (d.op == SHMEMX_OP_PUT || d.op == SHMEMX_OP_GET || d.op == SHMEMX_OP_PUT_SIGNAL) {
        exec_copy<false, true>(c, d, lo, hi, threadIdx.x, blockDim.x);
        if (__builtin_amdgcn_readfirstlane(d.op) == SHMEMX_OP_PUT_SIGNAL) {   // uniform: a barrier follows
            vshmem_detail::release_wg_at_exit();
            if (threadIdx.x == 0) signal_of(c, d);
        }
    }
}

// Ordering point between two phases of a batch, among the `units` work-groups
// of its grid; every thread calls it.  The count at `bar` only grows: arrival
// number old belongs to barrier old / units, and the one that completes it
// publishes the next number at VSHMEM_SYNC_GEN_OFF, on a line of its own,
// where the others wait.  With `units` fixed for the life of the words no
// reset separates a barrier from the next; the team barriers, whose callers
// may differ from phase to phase, must complete a store that resets the count
// before they can release anyone.  `g` is the number of the launch's next
// barrier; NONE before the first, whose arrival finds it.  Every work-group's
// stores are written back before its arrival (one release for all of its
// wavefronts, which have waited for their own), and every work-group
// invalidates after the wait.  The number is published without a release of
// its own, which would write the L2 back a second time: everything it stands
// for was in memory before the arrivals that it was counted from, the
// publisher's own stores with them, and nothing is stored in between.  (The
// language's memory model would want the release; the hardware's caches do
// not: a write-back has completed when the arrival's add is performed.)  A
// work-group that gives up a wait still arrives at every later barrier, so a
// launch that timed out leaves a whole number of barriers in the count.
constexpr uint64_t kNoBarrierYet = ~0ull;
__device__ __forceinline__ void phase_barrier(const shmemx_dctx_pub_t &c, uint64_t *bar, uint32_t units, uint64_t &g)
{
    vshmem_detail::wait_vm_complete();
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t *gen = (uint64_t *)((uint8_t *)bar + VSHMEM_SYNC_GEN_OFF);
        const uint64_t old = __hip_atomic_fetch_add(bar, 1ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        if (g == kNoBarrierYet) g = vshmem_detail::udiv(old, units);
        ++g;
        if (old + 1 == g * units) {
            vshmem_detail::acquire_agent();   // the other arrivals' releases
            __hip_atomic_store(gen, g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            vshmem_detail::spin_until<false>(c, gen, 3 /*GE*/, g);   // ends with an acquire
        }
    }
    __syncthreads();
}

}  // namespace vshmem_exec
