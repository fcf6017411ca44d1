/*
 * vshmem device API: device-initiated OpenSHMEM operations on virtual PEs
 * for gfx950 (MI355X).  HIP only; include from .hip sources.
 *
 * A kernel obtains the default device context (SHMEM_DEVICE_CTX_DEFAULT of
 * the paper's Section 6.2: created on the host at initialisation, published
 * GPU-visible, used by kernels, destroyed at finalisation) as a kernel
 * argument and binds it to the virtual PE the calling work-group acts for:
 *
 *     shmem_dctx_t ctx = shmemx_dctx_bind(published, blockIdx.x / wgs_per_pe);
 *
 * All pointer arguments are canonical symmetric addresses (PE 0's copy, as
 * returned by shmem_malloc); the library translates them with
 * addr(pe) = sym + pe * stride, without classifying pointers (Section 6.3).
 *
 * Scopes (Section 4.1, Section 6.3): a plain name is issued by one thread;
 * _wave by all 64 lanes of a wavefront; _wg by every thread of the
 * work-group; _grid by every work-group acting for the PE.  Every
 * participant passes identical arguments.
 *
 * Completion and ordering (Section 6.3, Section 6.4): a blocking put/get
 * returns at local completion (the source may be reused); remote
 * visibility needs shmem_quiet or a barrier.  shmem_fence orders the
 * caller's later operations after its earlier ones; shmem_quiet completes
 * the caller's operations device-wide (agent scope), which on this part
 * writes back dirty L2 lines so other XCDs observe them.  Atomics are
 * relaxed at agent scope: atomicity does not imply ordering.
 */
#ifndef VSHMEM_DEVICE_HPP
#define VSHMEM_DEVICE_HPP

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "vshmem.h"

/* ------------------------------------------------------------- contexts */
/* The published device context (one per library instance). */
struct shmemx_dctx_pub_t {
    uint8_t *base;               /* canonical base: PE 0's slice */
    uint64_t stride;             /* bytes between PE slices */
    uint64_t user_bytes;         /* allocatable bytes per PE */
    uint64_t scratch_off;        /* offset of the library scratch in a slice */
    uint32_t *err;               /* device error word */
    uint64_t wait_timeout_ticks; /* spin limit in wall-clock ticks */
    int32_t npes;
    int32_t debug;
};

/* A context bound to the virtual PE a caller acts for.  PE arguments of
 * the operations are numbered in the context's team: argument p names
 * world PE tstart + p * tstride.  The default context's team is the world
 * (identity numbering); an explicit context's team is the team it was
 * created from. */
struct shmem_dctx_t {
    shmemx_dctx_pub_t c;
    int32_t me;      /* world PE the caller acts for */
    int32_t idx;     /* its number in the context's team: shmem_my_pe */
    int32_t tstart;
    int32_t tstride;
    int32_t tsize;   /* shmem_n_pes */
    int32_t tslot;   /* the team's barrier words */
    int64_t options; /* SHMEM_CTX_* bits it was created with */
};

/* Device teams are shmemx_dteam_t of vshmem.h. */

/* An explicit device context as shmemx_device_ctx_create publishes it in
 * device memory (the explicit contexts of Section 6.2: created on the host,
 * passed to kernels as device-visible handles).  Read-only for kernels. */
struct shmemx_dctx_rec_t {
    shmemx_dctx_pub_t pub;
    shmemx_dteam_t team;
    int64_t options;
};

#define VSHMEM_SCRATCH_BYTES (64u << 10)
#define VSHMEM_SYNC_SLOT_BYTES 128u
#define VSHMEM_MAX_TEAMS 256
/* A barrier's arrival count is at scratch + slot * VSHMEM_SYNC_SLOT_BYTES and
 * its generation word VSHMEM_SYNC_GEN_OFF bytes further, in a second array
 * of slots: waiters poll the generation while arrivals add to the count, and
 * on one cache line the polls queue with the atomics. */
#define VSHMEM_SYNC_GEN_OFF (32u << 10)
static_assert(VSHMEM_MAX_TEAMS * VSHMEM_SYNC_SLOT_BYTES <= VSHMEM_SYNC_GEN_OFF &&
                  VSHMEM_SYNC_GEN_OFF + VSHMEM_MAX_TEAMS * VSHMEM_SYNC_SLOT_BYTES <= VSHMEM_SCRATCH_BYTES,
              "barrier counts and generations fit the scratch tail");

/* The default context (SHMEM_DEVICE_CTX_DEFAULT) for world PE `me`. */
__device__ __forceinline__ shmem_dctx_t shmemx_dctx_bind(const shmemx_dctx_pub_t &pub, int me)
{
    shmem_dctx_t c;
    c.c = pub;
    c.me = me;
    c.idx = me;
    c.tstart = 0;
    c.tstride = 1;
    c.tsize = pub.npes;
    c.tslot = 0;
    c.options = 0;
    return c;
}

/* An explicit context for its team's member `idx` (0 <= idx < team size). */
__device__ __forceinline__ shmem_dctx_t shmemx_dctx_bind_explicit(const shmemx_dctx_rec_t &rec, int idx)
{
    shmem_dctx_t c;
    c.c = rec.pub;
    c.me = rec.team.start + idx * rec.team.stride;
    c.idx = idx;
    c.tstart = rec.team.start;
    c.tstride = rec.team.stride;
    c.tsize = rec.team.size;
    c.tslot = rec.team.slot;
    c.options = rec.options;
    return c;
}

__device__ __forceinline__ int shmem_my_pe(const shmem_dctx_t &ctx) { return ctx.idx; }
__device__ __forceinline__ int shmem_n_pes(const shmem_dctx_t &ctx) { return ctx.tsize; }

/* The context's team as a device team descriptor. */
__device__ __forceinline__ shmemx_dteam_t shmemx_ctx_team(const shmem_dctx_t &ctx)
{
    return shmemx_dteam_t{ctx.tstart, ctx.tstride, ctx.tsize, ctx.tslot};
}

/* PE `pe`'s copy of a symmetric object, pe numbered in the context's team:
 * the device-domain shmem_ptr. */
template <typename T>
__device__ __forceinline__ T *shmem_ptr(const shmem_dctx_t &ctx, const T *sym, int pe)
{
    return (T *)((uint8_t *)sym + (uint64_t)(ctx.tstart + pe * ctx.tstride) * ctx.c.stride);
}

/* The caller's own copy of a symmetric object. */
template <typename T>
__device__ __forceinline__ T *shmemx_local_ptr(const shmem_dctx_t &ctx, const T *sym)
{
    return (T *)((uint8_t *)sym + (uint64_t)ctx.me * ctx.c.stride);
}

__device__ __forceinline__ int shmemx_team_pe(const shmemx_dteam_t &t, int k) { return t.start + k * t.stride; }

/* --------------------------------------------------------------- details */
namespace vshmem_detail {

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint64_t now() { return wall_clock64(); }

__device__ __forceinline__ uint64_t first_lane64(uint64_t x)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ void latch_error(const shmemx_dctx_pub_t &c, uint32_t bits)
{
    __hip_atomic_fetch_or(c.err, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void release_agent() { __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent"); }
/* Wait until this thread's earlier vector memory operations have completed
 * (stores acknowledged by L2): vmcnt(0), with the export and LDS counters
 * left alone.  Followed by a work-group barrier and one agent-scope release
 * by a single thread, it gives the whole work-group's stores agent-scope
 * visibility with one L2 write-back instead of one per wavefront. */
__device__ __forceinline__ void wait_vm_complete()
{
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

/* Agent-scope release of everything the work-group stored, with one L2
 * write-back: every thread waits for its own operations, the work-group
 * synchronises, thread 0 releases.  Every thread of the work-group must
 * call it.  An agent release per wavefront costs one write-back each, and
 * those serialise in the L2s (thousands of wavefronts: hundreds of us). */
__device__ __forceinline__ void release_wg_at_exit()
{
    wait_vm_complete();
    __syncthreads();
    if (threadIdx.x == 0) release_agent();
}
/* As above, and no thread returns before the release is done. */
__device__ __forceinline__ void release_wg()
{
    release_wg_at_exit();
    __syncthreads();
}
__device__ __forceinline__ void acquire_agent() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent"); }

template <bool NT, typename T>
__device__ __forceinline__ T ld(const T *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <bool NT, typename T>
__device__ __forceinline__ void st(T *p, T v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

/* Vector body: lane handles elements lane, lane+nl, ...; U loads are issued
 * before their stores so each lane keeps U*sizeof(V) bytes in flight. */
template <typename V, int U, bool NT>
__device__ __forceinline__ void copy_body(V *__restrict__ d, const V *__restrict__ s, uint64_t nv,
                                          uint64_t lane, uint64_t nl)
{
    uint64_t i = lane;
    for (; i + (uint64_t)(U - 1) * nl < nv; i += (uint64_t)U * nl) {
        V r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = ld<NT>(s + i + (uint64_t)u * nl);
#pragma unroll
        for (int u = 0; u < U; ++u) st<NT>(d + i + (uint64_t)u * nl, r[u]);
    }
    for (; i < nv; i += nl) st<NT>(d + i, ld<NT>(s + i));
}

/* A T at any address: gfx950 reads and writes global memory at any byte
 * address (unaligned access mode, the platform's default), so these are one
 * instruction, as for an aligned T. */
template <bool NT, typename T>
__device__ __forceinline__ T ld_any(const uint8_t *p)
{
    typedef T A __attribute__((aligned(1)));
    if constexpr (NT) return __builtin_nontemporal_load((const A *)p);
    else return *(const A *)p;
}

template <bool NT, typename T>
__device__ __forceinline__ void st_any(uint8_t *p, T v)
{
    typedef T A __attribute__((aligned(1)));
    if constexpr (NT) __builtin_nontemporal_store(v, (A *)p);
    else *(A *)p = v;
}

/* The loads before this line are issued before it: the compiler would sink
 * a load whose value only a conditional store uses into the condition. */
__device__ __forceinline__ void loads_issued() { asm volatile("" ::: "memory"); }

/* The same for loads through a __restrict__ pointer, which an asm statement
 * that does not name them would not keep: all of them have arrived here. */
template <int V>
__device__ __forceinline__ void loaded(v4u (&r)[V])
{
    static_assert(V <= 4 || V == 8, "");
    if constexpr (V == 2) asm volatile("" : "+v"(r[0]), "+v"(r[1]));
    if constexpr (V == 3) asm volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]));
    if constexpr (V == 4) asm volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]));
    if constexpr (V == 8)
        asm volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]), "+v"(r[4]), "+v"(r[5]), "+v"(r[6]), "+v"(r[7]));
}

/* Up to K pieces of 16 bytes from o on by one lane, the last one ending at the
 * last byte; cnt of them are this lane's. */
template <int K, bool NT>
__device__ __forceinline__ void lone_rest(uint8_t *__restrict__ d, const uint8_t *__restrict__ s, uint64_t n, uint64_t o,
                                          uint32_t cnt)
{
    v4u r[K];
#pragma unroll
    for (int u = 0; u < K; ++u) r[u] = ld_any<NT, v4u>(s + min(o + 16 * u, n - 16));
    loaded(r);
#pragma unroll
    for (int u = 0; u < K; ++u)
        if (u == 0 || u < cnt) st_any<NT, v4u>(d + min(o + 16 * u, n - 16), r[u]);
}

/* Copy of n bytes by one lane.  Below 16 bytes, two pieces of the widest size
 * that fits, the second ending at the last byte (one when it fits exactly: an
 * 8-byte message is one 8-byte move).  Longer ones: 16 U bytes at a time, on
 * the destination's boundaries when there is more than that, and the rest in
 * one round trip, with as many loads as the wavefront's longest rest needs:
 * lanes with messages of different lengths wait once, and no lane of many
 * with one length loads a piece twice, 64 lanes reading 64 messages being 64
 * lines each time (64 PEs x 1024 lanes, 4096 messages of 16 bytes per PE: 8.3
 * us with four pieces always in flight, 6.6 so). */
template <int U, bool NT>
__device__ __forceinline__ void copy_lone(uint8_t *__restrict__ d, const uint8_t *__restrict__ s, uint64_t n)
{
    static_assert(U <= 4, "");
    if (n < 16) {
        if (n >= 8) {
            const uint64_t a = ld_any<NT, uint64_t>(s), b = ld_any<NT, uint64_t>(s + n - 8);
            st_any<NT, uint64_t>(d, a);
            if (n > 8) st_any<NT, uint64_t>(d + n - 8, b);
        } else if (n >= 4) {
            const uint32_t a = ld_any<NT, uint32_t>(s), b = ld_any<NT, uint32_t>(s + n - 4);
            st_any<NT, uint32_t>(d, a);
            if (n > 4) st_any<NT, uint32_t>(d + n - 4, b);
        } else if (n >= 2) {
            const uint16_t a = ld_any<NT, uint16_t>(s), b = ld_any<NT, uint16_t>(s + n - 2);
            st_any<NT, uint16_t>(d, a);
            if (n > 2) st_any<NT, uint16_t>(d + n - 2, b);
        } else if (n) {
            *d = *s;
        }
        return;
    }
    uint64_t o = 0;
    if (n > 16 * U) {
        o = (16 - ((uintptr_t)d & 15)) & 15;
        if (o) st_any<NT, v4u>(d, ld_any<NT, v4u>(s));
        for (; o + 16 * U <= n; o += 16 * U) {
            v4u r[U];
#pragma unroll
            for (int u = 0; u < U; ++u) r[u] = ld_any<NT, v4u>(s + o + 16 * u);
#pragma unroll
            for (int u = 0; u < U; ++u) st_any<NT, v4u>(d + o + 16 * u, r[u]);
        }
        if (o >= n) return;
    }
    const uint32_t cnt = ((uint32_t)(n - o) + 15) >> 4;   // 1 to U
    if (U > 3 && __ballot(cnt > 3)) lone_rest<4, NT>(d, s, n, o, cnt);
    else if (U > 2 && __ballot(cnt > 2)) lone_rest<3, NT>(d, s, n, o, cnt);
    else if (U > 1 && __ballot(cnt > 1)) lone_rest<2, NT>(d, s, n, o, cnt);
    else lone_rest<1, NT>(d, s, n, o, cnt);
}

/* Pieces 0 .. np - 1 of 16 bytes by nl lanes, V in flight per lane (of whole
 * wavefronts: each takes one contiguous run): piece k at 16 k, at most at
 * `last` (which may lie before 0), and piece np - 1 at `end`.  np is at most
 * V nl; with MORE it may be one more, which lane 0 takes; with LOOP any number.
 * Lanes past the end load a piece again and no load is under a condition of
 * its own: after a conditional load the compiler puts a wait, a round trip for
 * each. */
enum { FIT, MORE, LOOP };
template <int V, bool NT, int KIND>
__device__ __forceinline__ void copy_pieces(uint8_t *__restrict__ d, const uint8_t *__restrict__ s, uint64_t np,
                                            int64_t last, int64_t end, uint64_t lane, uint64_t nl)
{
    const bool waves = (nl & 63) == 0;
    const uint64_t w = waves ? 64 : nl;
    uint64_t k = waves ? (lane >> 6) * (V * 64) + (lane & 63) : lane;
    if (k >= np) return;
    auto at = [&](int v) {
        const uint64_t q = k + v * w;
        return q + 1 >= np ? end : min((int64_t)(16 * q), last);
    };
    do {
        // (The places are computed where they are used: for the stores anew, and
        // not ahead of a loop over messages.  Kept, they take four registers each.)
        asm volatile("" : "+v"(k));
        v4u r[V], x;
#pragma unroll
        for (int v = 0; v < V; ++v) r[v] = ld_any<NT, v4u>(s + at(v));
        const bool more = KIND == MORE && np > V * nl;
        if (more) x = ld_any<NT, v4u>(s + end);
        loaded(r);
        asm volatile("" : "+v"(k));
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (v == 0 || k + v * w < np) st_any<NT, v4u>(d + at(v), r[v]);
        if (more && lane == 0) st_any<NT, v4u>(d + end, x);
        k += V * nl;
    } while (KIND == LOOP && k < np);
}

/* Copy n bytes with nl cooperating lanes (this one is `lane`), at any
 * alignment of either side.  n >= 16: the destination's 16-byte vectors that
 * lie inside the message (stores stay aligned, loads take the source as it
 * falls), and the first and the last 16 bytes where the destination's edges
 * are not on a boundary; those overlap the vectors beside them and write the
 * same bytes.  LONE marks a copy by one lane (lane 0 of 1).  R is the number of
 * pieces a lane keeps in flight in the remainder, U or less.  Without SHORT a
 * short message takes the longer ones' way: the batches' executors, which run
 * a few messages of all lengths each, are better off with less code (2000
 * operations on 64 PEs with completion stamps: 29 us so, 32 with both ways).
 *
 * Bound by HBM for large messages, by a round trip and the instructions around
 * it for short ones: so one piece per lane where the lanes suffice, whatever
 * the alignment, and no loop.  A user's kernel putting one message after
 * another, 4096 per PE, 64 PEs x 4 work-groups of 256: by wavefronts 64 bytes
 * 92 us, where edges of their own and a conditional load per vector took 145;
 * 1501 bytes at odd addresses 288; by work-groups 16 bytes 334 (515), 1 KiB 645
 * (857).  With one wavefront per message, one message at a time, 1501 bytes at
 * addresses that disagree modulo 16 moved at 2.6 TB/s, against 0.44 with
 * elements down to bytes.  16 MiB messages by 1024 threads, aligned, U = 8:
 * 6.1 TB/s, against 5.7 with every nl-th vector instead of contiguous runs per
 * wavefront.  What is left behind aligned vectors joined by funnel shifts:
 * sources off a boundary, 16 and 32 KiB by 1024 threads, 247 us and 217. */
template <int U, bool NT, bool LONE = false, int R = U, bool SHORT = true>
__device__ __forceinline__ void copy_bytes(uint8_t *__restrict__ d, const uint8_t *__restrict__ s, uint64_t n,
                                           uint64_t lane, uint64_t nl)
{
    if constexpr (LONE) {
        copy_lone<U, NT>(d, s, n);
        return;
    }
    if (n < 16) {
        for (uint64_t i = lane; i < n; i += nl) d[i] = s[i];
        return;
    }
    // The destination's vectors that hold bytes of the message, moved inward
    // to lie inside it: one piece per lane where the lanes suffice.
    const uint64_t mis = (uintptr_t)d & 15, np = (mis + n + 15) >> 4;
    if (SHORT && np <= nl) {
        if (lane < np) {
            const uint64_t o = min(lane ? 16 * lane - mis : 0, n - 16);
            st_any<NT, v4u>(d + o, ld_any<NT, v4u>(s + o));
        }
        return;
    }
    const uint64_t head = (16 - mis) & 15, nv = (n - head) / 16;
    // Full batches: a wavefront's U vectors per lane are one contiguous run
    // (whole wavefronts; other lane counts take every nl-th vector).  With a
    // source that is not on a boundary each wavefront then reads its lines
    // once, but for the last: 64 KiB messages at odd addresses by 1024
    // threads moved at 5.6 TB/s, and at 4.6 with every nl-th vector.
    const bool waves = (nl & 63) == 0;
    const uint64_t w = waves ? 64 : nl;
    uint64_t first = waves ? (lane >> 6) * (U * 64) + (lane & 63) : lane;
    if (R == U) asm volatile("" : "+v"(first));   // (as in copy_pieces; k_pairs 92 registers without, 76 with)
    v4u *dv = (v4u *)(d + head);
    const uint8_t *sv = s + head;
    uint64_t nb = 0;
    for (; nb + U * nl <= nv; nb += U * nl) {
        const uint64_t i = nb + first;
        v4u r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = ld_any<NT, v4u>(sv + 16 * (i + u * w));
#pragma unroll
        for (int u = 0; u < U; ++u) st<NT>(dv + i + u * w, r[u]);
    }
    // The rest, in one round trip (R = U): the vectors past the batches, the last 16
    // bytes if the end is off a boundary, and as the last piece the first 16
    // bytes if the start is.
    const uint64_t rest = np - nb;
    if (rest == 0) return;
    const uint64_t at = head + 16 * nb;
    const int64_t last = (int64_t)(n - 16 - at), end = head ? -(int64_t)at : last;
    d += at;
    s += at;
    if (SHORT && U > 1 && rest <= nl) copy_pieces<1, NT, FIT>(d, s, rest, last, end, lane, nl);
    else if (SHORT && U > 2 && R <= 4 && rest <= 2 * nl) copy_pieces<2, NT, FIT>(d, s, rest, last, end, lane, nl);
    else if (R > 4 && rest <= 4 * nl) copy_pieces<4, NT, FIT>(d, s, rest, last, end, lane, nl);
    else copy_pieces<R, NT, R == U ? MORE : LOOP>(d, s, rest, last, end, lane, nl);
}

__device__ __forceinline__ bool cmp_holds_u(uint64_t x, int cmp, uint64_t v)
{
    switch (cmp) {
    case 0: return x == v;
    case 1: return x != v;
    case 2: return x > v;
    case 3: return x >= v;
    case 4: return x < v;
    default: return x <= v;
    }
}

__device__ __forceinline__ bool cmp_holds_s(int64_t x, int cmp, int64_t v)
{
    switch (cmp) {
    case 0: return x == v;
    case 1: return x != v;
    case 2: return x > v;
    case 3: return x >= v;
    case 4: return x < v;
    default: return x <= v;
    }
}

/* Spin until the 64-bit word satisfies cmp, with backoff and a spin limit;
 * returns the last value read.  Latches a device error on timeout. */
template <bool SIGNED>
__device__ __forceinline__ uint64_t spin_until(const shmemx_dctx_pub_t &c, uint64_t *w, int cmp, uint64_t v)
{
    uint64_t x = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool ok = SIGNED ? cmp_holds_s((int64_t)x, cmp, (int64_t)v) : cmp_holds_u(x, cmp, v);
    if (!ok) {
        uint64_t t0 = now();
        for (;;) {
            __builtin_amdgcn_s_sleep(1);
            x = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ok = SIGNED ? cmp_holds_s((int64_t)x, cmp, (int64_t)v) : cmp_holds_u(x, cmp, v);
            if (ok) break;
            if (now() - t0 > c.wait_timeout_ticks) {
                latch_error(c, 0x1u);
                break;
            }
        }
    }
    acquire_agent();
    return x;
}

__device__ __forceinline__ uint64_t *sync_slot(const shmemx_dctx_pub_t &c, int pe, int slot)
{
    return (uint64_t *)(c.base + (uint64_t)pe * c.stride + c.scratch_off + (uint64_t)slot * VSHMEM_SYNC_SLOT_BYTES);
}

/* Counter barrier among `units` arriving work-groups; one thread per
 * work-group calls it.  The arrival word holds the phase number (high 32
 * bits) and the arrivals of the phase so far (low 32 bits); the generation
 * word, VSHMEM_SYNC_GEN_OFF further on a line of its own, holds the number
 * of completed phases.  An arrival learns its phase from its own fetch_add
 * and waits until the generation reaches phase + 1; the last arrival
 * resets the count with the next phase number and then releases the
 * generation.  No separate read of the generation precedes the arrival: on
 * a line of its own such a read can complete after the arrival, see the
 * next generation, and wait for a phase that needs its own arrival.
 * Release before arriving, acquire after leaving (in both the last arrival
 * and the waiters), so it also completes (quiets) the arrivals' stores.
 * Called after the work-group's threads waited for their own operations
 * and synchronised, the release and acquire of this one thread cover the
 * whole work-group: they write back and invalidate the caches the
 * work-group's wavefronts share.  With the generation word on a line of
 * its own a 64-PE barrier took 3.2 us instead of 5.9, a 256-PE one 9.5
 * instead of 21.5 (waiters' polls no longer queue with the arrivals'
 * atomics).  `meanwhile` runs between the arrival and the wait. */
struct Nothing {
    __device__ __forceinline__ void operator()() const {}
};
template <class F = Nothing>
__device__ __forceinline__ void counter_barrier(const shmemx_dctx_pub_t &c, uint64_t *slot, uint64_t units,
                                                F meanwhile = F())
{
    uint64_t *cnt = slot;
    uint64_t *gen = (uint64_t *)((uint8_t *)slot + VSHMEM_SYNC_GEN_OFF);
    release_agent();
    const uint64_t old = __hip_atomic_fetch_add(cnt, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t next = (uint64_t)((uint32_t)(old >> 32) + 1u);
    const bool last = (old & 0xffffffffull) == units - 1;
    if (last) {
        acquire_agent();   // the other arrivals' releases
        __hip_atomic_store(cnt, next << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(gen, next, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
    meanwhile();
    if (!last) spin_until<false>(c, gen, 0 /*EQ*/, next);
    acquire_agent();
}

} // namespace vshmem_detail

/* ---------------------------------------------------------- debug checks */
/* Contexts published with debug set (VSHMEM_DEBUG at init) check every
 * operation's arguments: operands inside PE 0's user heap (canonical
 * symmetric addresses), 8-byte words aligned, PE numbers inside the
 * context's team, and for _wave/_wg/_grid calls one argument set across the
 * participants.  A failed check latches SHMEMX_DEVERR_BAD_ADDRESS or
 * SHMEMX_DEVERR_NONUNIFORM and the operation does nothing (every
 * participant of a scoped call takes the same decision).  Without debug the
 * checks reduce to one uniform branch. */
namespace vshmem_detail {

__device__ __forceinline__ bool in_user_heap(const shmem_dctx_t &ctx, const void *p, uint64_t n)
{
    const uint8_t *q = (const uint8_t *)p;
    if (q < ctx.c.base) return false;
    const uint64_t off = (uint64_t)(q - ctx.c.base);
    return off <= ctx.c.user_bytes && n <= ctx.c.user_bytes - off;
}

__device__ __forceinline__ bool pe_in_team(const shmem_dctx_t &ctx, int pe) { return pe >= 0 && pe < ctx.tsize; }

__device__ __forceinline__ bool checked(const shmem_dctx_t &ctx, bool ok)
{
    if (!ok) latch_error(ctx.c, SHMEMX_DEVERR_BAD_ADDRESS);
    return ok;
}

/* A put or get of n bytes with PE pe (both operands symmetric). */
__device__ __forceinline__ bool rma_ok(const shmem_dctx_t &ctx, const void *dest, const void *src, uint64_t n, int pe)
{
    return !ctx.c.debug || checked(ctx, in_user_heap(ctx, dest, n) && in_user_heap(ctx, src, n) && pe_in_team(ctx, pe));
}

/* A naturally aligned symmetric 8-byte word on PE pe. */
__device__ __forceinline__ bool word_ok(const shmem_dctx_t &ctx, const void *w, int pe)
{
    return !ctx.c.debug || checked(ctx, ((uintptr_t)w & 7) == 0 && in_user_heap(ctx, w, 8) && pe_in_team(ctx, pe));
}

/* Wavefront scope: every lane passed lane 0's arguments and found them
 * valid.  All lanes return the same answer. */
__device__ __forceinline__ bool wave_agree(const shmem_dctx_t &ctx, bool ok, uint64_t a, uint64_t b, uint64_t c,
                                           uint64_t d)
{
    if (!ctx.c.debug) return true;
    const bool same = a == first_lane64(a) && b == first_lane64(b) && c == first_lane64(c) && d == first_lane64(d);
    if (__ballot(!same) != 0 && __lane_id() == 0) latch_error(ctx.c, SHMEMX_DEVERR_NONUNIFORM);
    return __ballot(!(ok && same)) == 0;
}

/* Work-group scope: the same through LDS.  Every thread must call it. */
__device__ __forceinline__ bool wg_agree(const shmem_dctx_t &ctx, bool ok, uint64_t a, uint64_t b, uint64_t c,
                                         uint64_t d)
{
    if (!ctx.c.debug) return true;
    __shared__ uint64_t ref[4];
    __shared__ uint32_t verdict;   // bit 0: a thread found its arguments invalid; bit 1: arguments differ
    if (threadIdx.x == 0) {
        ref[0] = a;
        ref[1] = b;
        ref[2] = c;
        ref[3] = d;
        verdict = 0;
    }
    __syncthreads();
    const bool same = a == ref[0] && b == ref[1] && c == ref[2] && d == ref[3];
    if (!ok || !same) atomicOr(&verdict, (ok ? 0u : 1u) | (same ? 0u : 2u));
    __syncthreads();
    const uint32_t v = __builtin_amdgcn_readfirstlane(verdict);
    __syncthreads();   // ref and verdict are free for the next call
    if ((v & 2u) && threadIdx.x == 0) latch_error(ctx.c, SHMEMX_DEVERR_NONUNIFORM);
    return v == 0;
}

} // namespace vshmem_detail

#define VSHMEM_U64(x) ((uint64_t)(uintptr_t)(x))

/* ------------------------------------------------------------ put / get */
#define VSHMEM_COPY_UNROLL 4

/* put: PE `pe`'s dest[0, n) <- my src[0, n) */
__device__ __forceinline__ void shmem_putmem(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    if (!vshmem_detail::rma_ok(ctx, dest, src, n, pe)) return;
    vshmem_detail::copy_bytes<VSHMEM_COPY_UNROLL, false, true>(shmem_ptr(ctx, (uint8_t *)dest, pe),
                                                               shmemx_local_ptr(ctx, (const uint8_t *)src), n, 0, 1);
}
__device__ __forceinline__ void shmem_putmem_nbi(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_putmem(ctx, dest, src, n, pe);
}
__device__ __forceinline__ void shmem_putmem_wave(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    if (!vshmem_detail::wave_agree(ctx, vshmem_detail::rma_ok(ctx, dest, src, n, pe), VSHMEM_U64(dest),
                                   VSHMEM_U64(src), n, (uint64_t)pe))
        return;
    vshmem_detail::copy_bytes<VSHMEM_COPY_UNROLL, false>(shmem_ptr(ctx, (uint8_t *)dest, pe),
                                                         shmemx_local_ptr(ctx, (const uint8_t *)src), n,
                                                         __lane_id(), 64);
}
__device__ __forceinline__ void shmem_putmem_nbi_wave(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_putmem_wave(ctx, dest, src, n, pe);
}
__device__ __forceinline__ void shmem_putmem_nbi_wg(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    if (!vshmem_detail::wg_agree(ctx, vshmem_detail::rma_ok(ctx, dest, src, n, pe), VSHMEM_U64(dest), VSHMEM_U64(src),
                                 n, (uint64_t)pe))
        return;
    vshmem_detail::copy_bytes<VSHMEM_COPY_UNROLL, false>(shmem_ptr(ctx, (uint8_t *)dest, pe),
                                                         shmemx_local_ptr(ctx, (const uint8_t *)src), n,
                                                         threadIdx.x, blockDim.x);
}
__device__ __forceinline__ void shmem_putmem_wg(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_putmem_nbi_wg(ctx, dest, src, n, pe);
    __syncthreads();
}
/* Grid scope: the nwgs work-groups acting for the PE (this one is `rank`)
 * share the message; each returns when its own share is locally complete.
 * Debug checks compare arguments within each work-group. */
__device__ __forceinline__ void shmemx_putmem_grid(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n,
                                                   int pe, int rank, int nwgs)
{
    if (!vshmem_detail::wg_agree(ctx, vshmem_detail::rma_ok(ctx, dest, src, n, pe), VSHMEM_U64(dest), VSHMEM_U64(src),
                                 n, ((uint64_t)(uint32_t)nwgs << 32) | (uint32_t)pe))
        return;
    vshmem_detail::copy_bytes<VSHMEM_COPY_UNROLL, false>(shmem_ptr(ctx, (uint8_t *)dest, pe),
                                                         shmemx_local_ptr(ctx, (const uint8_t *)src), n,
                                                         (uint64_t)rank * blockDim.x + threadIdx.x,
                                                         (uint64_t)nwgs * blockDim.x);
}

/* get: my dest[0, n) <- PE `pe`'s src[0, n) */
__device__ __forceinline__ void shmem_getmem(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    if (!vshmem_detail::rma_ok(ctx, dest, src, n, pe)) return;
    vshmem_detail::copy_bytes<VSHMEM_COPY_UNROLL, false, true>(shmemx_local_ptr(ctx, (uint8_t *)dest),
                                                               shmem_ptr(ctx, (const uint8_t *)src, pe), n, 0, 1);
}
__device__ __forceinline__ void shmem_getmem_nbi(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_getmem(ctx, dest, src, n, pe);
}
__device__ __forceinline__ void shmem_getmem_wave(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    if (!vshmem_detail::wave_agree(ctx, vshmem_detail::rma_ok(ctx, dest, src, n, pe), VSHMEM_U64(dest),
                                   VSHMEM_U64(src), n, (uint64_t)pe))
        return;
    vshmem_detail::copy_bytes<VSHMEM_COPY_UNROLL, false>(shmemx_local_ptr(ctx, (uint8_t *)dest),
                                                         shmem_ptr(ctx, (const uint8_t *)src, pe), n,
                                                         __lane_id(), 64);
}
__device__ __forceinline__ void shmem_getmem_nbi_wave(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_getmem_wave(ctx, dest, src, n, pe);
}
__device__ __forceinline__ void shmem_getmem_nbi_wg(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    if (!vshmem_detail::wg_agree(ctx, vshmem_detail::rma_ok(ctx, dest, src, n, pe), VSHMEM_U64(dest), VSHMEM_U64(src),
                                 n, (uint64_t)pe))
        return;
    vshmem_detail::copy_bytes<VSHMEM_COPY_UNROLL, false>(shmemx_local_ptr(ctx, (uint8_t *)dest),
                                                         shmem_ptr(ctx, (const uint8_t *)src, pe), n,
                                                         threadIdx.x, blockDim.x);
}
__device__ __forceinline__ void shmem_getmem_wg(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_getmem_nbi_wg(ctx, dest, src, n, pe);
    __syncthreads();
}
__device__ __forceinline__ void shmemx_getmem_grid(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n,
                                                   int pe, int rank, int nwgs)
{
    if (!vshmem_detail::wg_agree(ctx, vshmem_detail::rma_ok(ctx, dest, src, n, pe), VSHMEM_U64(dest), VSHMEM_U64(src),
                                 n, ((uint64_t)(uint32_t)nwgs << 32) | (uint32_t)pe))
        return;
    vshmem_detail::copy_bytes<VSHMEM_COPY_UNROLL, false>(shmemx_local_ptr(ctx, (uint8_t *)dest),
                                                         shmem_ptr(ctx, (const uint8_t *)src, pe), n,
                                                         (uint64_t)rank * blockDim.x + threadIdx.x,
                                                         (uint64_t)nwgs * blockDim.x);
}

/* GPU-space names.  The paper's GPU-space usage example (Section 6.1) writes
 * a device-initiated put to an object from shmemg_malloc as shmemg_put and
 * marks its names as illustrative.  Here the GPU space is the default heap,
 * so these are the put and get above under that prefix. */
__device__ __forceinline__ void shmemg_putmem(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_putmem(ctx, dest, src, n, pe);
}
__device__ __forceinline__ void shmemg_putmem_nbi(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_putmem_nbi(ctx, dest, src, n, pe);
}
__device__ __forceinline__ void shmemg_putmem_wave(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_putmem_wave(ctx, dest, src, n, pe);
}
__device__ __forceinline__ void shmemg_putmem_wg(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_putmem_wg(ctx, dest, src, n, pe);
}
__device__ __forceinline__ void shmemg_getmem(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_getmem(ctx, dest, src, n, pe);
}
__device__ __forceinline__ void shmemg_getmem_nbi(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_getmem_nbi(ctx, dest, src, n, pe);
}
__device__ __forceinline__ void shmemg_getmem_wave(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_getmem_wave(ctx, dest, src, n, pe);
}
__device__ __forceinline__ void shmemg_getmem_wg(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n, int pe)
{
    shmem_getmem_wg(ctx, dest, src, n, pe);
}

/* -------------------------------------------------------- fence / quiet */
__device__ __forceinline__ void shmem_fence(const shmem_dctx_t &) { vshmem_detail::release_agent(); }
__device__ __forceinline__ void shmem_quiet(const shmem_dctx_t &) { vshmem_detail::release_agent(); }
__device__ __forceinline__ void shmem_quiet_wave(const shmem_dctx_t &) { vshmem_detail::release_agent(); }
__device__ __forceinline__ void shmem_fence_wave(const shmem_dctx_t &) { vshmem_detail::release_agent(); }
/* Every lane completes its own stores, then the work-group synchronises:
 * all of the work-group's earlier operations are complete on return. */
__device__ __forceinline__ void shmem_quiet_wg(const shmem_dctx_t &) { vshmem_detail::release_wg(); }
__device__ __forceinline__ void shmem_fence_wg(const shmem_dctx_t &ctx) { shmem_quiet_wg(ctx); }

/* --------------------------------------------------------------- atomics */
#define VSHMEM_AMO_PTR(T) ((T *)shmem_ptr(ctx, (uint8_t *)dest, pe))

__device__ __forceinline__ int64_t shmem_int64_atomic_fetch_add(const shmem_dctx_t &ctx, int64_t *dest, int64_t v, int pe)
{
    if (!vshmem_detail::word_ok(ctx, dest, pe)) return 0;
    return (int64_t)__hip_atomic_fetch_add(VSHMEM_AMO_PTR(uint64_t), (uint64_t)v, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void shmem_int64_atomic_add(const shmem_dctx_t &ctx, int64_t *dest, int64_t v, int pe)
{
    if (!vshmem_detail::word_ok(ctx, dest, pe)) return;
    __hip_atomic_fetch_add(VSHMEM_AMO_PTR(uint64_t), (uint64_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t shmem_uint64_atomic_fetch_xor(const shmem_dctx_t &ctx, uint64_t *dest, uint64_t v, int pe)
{
    if (!vshmem_detail::word_ok(ctx, dest, pe)) return 0;
    return __hip_atomic_fetch_xor(VSHMEM_AMO_PTR(uint64_t), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int64_t shmem_int64_atomic_fetch_xor(const shmem_dctx_t &ctx, int64_t *dest, int64_t v, int pe)
{
    if (!vshmem_detail::word_ok(ctx, dest, pe)) return 0;
    return (int64_t)__hip_atomic_fetch_xor(VSHMEM_AMO_PTR(uint64_t), (uint64_t)v, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void shmem_uint64_atomic_xor(const shmem_dctx_t &ctx, uint64_t *dest, uint64_t v, int pe)
{
    if (!vshmem_detail::word_ok(ctx, dest, pe)) return;
    __hip_atomic_fetch_xor(VSHMEM_AMO_PTR(uint64_t), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void shmem_int64_atomic_xor(const shmem_dctx_t &ctx, int64_t *dest, int64_t v, int pe)
{
    if (!vshmem_detail::word_ok(ctx, dest, pe)) return;
    __hip_atomic_fetch_xor(VSHMEM_AMO_PTR(uint64_t), (uint64_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int64_t shmem_int64_atomic_compare_swap(const shmem_dctx_t &ctx, int64_t *dest, int64_t cond,
                                                                   int64_t v, int pe)
{
    if (!vshmem_detail::word_ok(ctx, dest, pe)) return 0;
    uint64_t expected = (uint64_t)cond;
    __hip_atomic_compare_exchange_strong(VSHMEM_AMO_PTR(uint64_t), &expected, (uint64_t)v, __ATOMIC_RELAXED,
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (int64_t)expected;
}
__device__ __forceinline__ int64_t shmem_int64_atomic_fetch(const shmem_dctx_t &ctx, const int64_t *dest, int pe)
{
    if (!vshmem_detail::word_ok(ctx, dest, pe)) return 0;
    return (int64_t)__hip_atomic_load((uint64_t *)shmem_ptr(ctx, (const uint8_t *)dest, pe), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void shmem_int64_atomic_set(const shmem_dctx_t &ctx, int64_t *dest, int64_t v, int pe)
{
    if (!vshmem_detail::word_ok(ctx, dest, pe)) return;
    __hip_atomic_store(VSHMEM_AMO_PTR(uint64_t), (uint64_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int64_t shmem_int64_atomic_swap(const shmem_dctx_t &ctx, int64_t *dest, int64_t v, int pe)
{
    if (!vshmem_detail::word_ok(ctx, dest, pe)) return 0;
    return (int64_t)__hip_atomic_exchange(VSHMEM_AMO_PTR(uint64_t), (uint64_t)v, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
}

/* ------------------------------------------------- signals and waiting */
__device__ __forceinline__ void vshmemx_signal_update(const shmem_dctx_t &ctx, uint64_t *sig, uint64_t v, int sig_op, int pe)
{
    if (!vshmem_detail::word_ok(ctx, sig, pe)) return;
    uint64_t *s = shmem_ptr(ctx, sig, pe);
    if (sig_op == 1)
        __hip_atomic_fetch_add(s, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        __hip_atomic_store(s, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

/* put with signal: the data, a release, then the signal; the signal is
 * never observable before the data. */
__device__ __forceinline__ void shmem_putmem_signal(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n,
                                                    uint64_t *sig, uint64_t sigval, int sig_op, int pe)
{
    if (!vshmem_detail::word_ok(ctx, sig, pe) || !vshmem_detail::rma_ok(ctx, dest, src, n, pe)) return;
    shmem_putmem(ctx, dest, src, n, pe);
    vshmem_detail::release_agent();
    vshmemx_signal_update(ctx, sig, sigval, sig_op, pe);
}
__device__ __forceinline__ void shmem_putmem_signal_wave(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n,
                                                         uint64_t *sig, uint64_t sigval, int sig_op, int pe)
{
    const bool data_ok = vshmem_detail::wave_agree(ctx, vshmem_detail::rma_ok(ctx, dest, src, n, pe), VSHMEM_U64(dest),
                                                   VSHMEM_U64(src), n, (uint64_t)pe);
    const bool sig_ok = vshmem_detail::wave_agree(ctx, vshmem_detail::word_ok(ctx, sig, pe), VSHMEM_U64(sig), sigval,
                                                  (uint64_t)sig_op, (uint64_t)pe);
    if (!data_ok || !sig_ok) return;
    shmem_putmem_wave(ctx, dest, src, n, pe);
    vshmem_detail::release_agent();
    if (__lane_id() == 0) vshmemx_signal_update(ctx, sig, sigval, sig_op, pe);
}
__device__ __forceinline__ void shmem_putmem_signal_wg(const shmem_dctx_t &ctx, void *dest, const void *src, size_t n,
                                                       uint64_t *sig, uint64_t sigval, int sig_op, int pe)
{
    const bool data_ok = vshmem_detail::wg_agree(ctx, vshmem_detail::rma_ok(ctx, dest, src, n, pe), VSHMEM_U64(dest),
                                                 VSHMEM_U64(src), n, (uint64_t)pe);
    const bool sig_ok = vshmem_detail::wg_agree(ctx, vshmem_detail::word_ok(ctx, sig, pe), VSHMEM_U64(sig), sigval,
                                                (uint64_t)sig_op, (uint64_t)pe);
    if (!data_ok || !sig_ok) return;
    shmem_putmem_nbi_wg(ctx, dest, src, n, pe);
    vshmem_detail::release_wg_at_exit();
    if (threadIdx.x == 0) vshmemx_signal_update(ctx, sig, sigval, sig_op, pe);
    __syncthreads();
}

/* Wait on my own copy of a symmetric uint64 signal. */
__device__ __forceinline__ uint64_t shmem_signal_wait_until(const shmem_dctx_t &ctx, uint64_t *sig, int cmp, uint64_t v)
{
    if (!vshmem_detail::word_ok(ctx, sig, ctx.idx)) return 0;
    return vshmem_detail::spin_until<false>(ctx.c, shmemx_local_ptr(ctx, sig), cmp, v);
}
__device__ __forceinline__ void shmem_int64_wait_until(const shmem_dctx_t &ctx, int64_t *ivar, int cmp, int64_t v)
{
    if (!vshmem_detail::word_ok(ctx, ivar, ctx.idx)) return;
    vshmem_detail::spin_until<true>(ctx.c, (uint64_t *)shmemx_local_ptr(ctx, ivar), cmp, (uint64_t)v);
}
__device__ __forceinline__ int shmem_int64_test(const shmem_dctx_t &ctx, int64_t *ivar, int cmp, int64_t v)
{
    if (!vshmem_detail::word_ok(ctx, ivar, ctx.idx)) return 0;
    int64_t x = (int64_t)__hip_atomic_load((uint64_t *)shmemx_local_ptr(ctx, ivar), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
    bool ok = vshmem_detail::cmp_holds_s(x, cmp, v);
    if (ok) vshmem_detail::acquire_agent();
    return ok ? 1 : 0;
}
/* Work-group scope wait: thread 0 spins, everyone acquires. */
__device__ __forceinline__ uint64_t shmem_signal_wait_until_wg(const shmem_dctx_t &ctx, uint64_t *sig, int cmp, uint64_t v)
{
    __shared__ uint64_t seen;
    if (threadIdx.x == 0) seen = shmem_signal_wait_until(ctx, sig, cmp, v);
    __syncthreads();
    vshmem_detail::acquire_agent();
    return seen;
}

/* ------------------------------------------------------------- barriers */
/* Team barriers (Section 6.3: barriers among the device-initiated
 * collectives; the scope suffix names who calls, as in the _wave example
 * of Section 8).  No member leaves before every member arrived, and each
 * caller's earlier operations are complete and visible device-wide on
 * return (the barrier implies quiet).  The counter lives in the scratch
 * tail of the team's first member, at the team's slot.
 *
 *   plain  one thread acts for its PE (exactly one per member calls);
 *   _wave  all 64 lanes of one wavefront act for the PE;
 *   _wg    every thread of one work-group acts for the PE;
 *   units  every thread of `units_per_pe` work-groups per PE.
 *
 * All callers of one barrier must be resident together: a caller that is
 * waiting for a work-group slot never arrives. */
__device__ __forceinline__ void shmemx_team_sync_units(const shmem_dctx_t &ctx, const shmemx_dteam_t &team,
                                                       uint64_t units_per_pe)
{
    // Every thread's operations complete before the work-group arrives;
    // thread 0's release and acquire inside the barrier then cover them all.
    vshmem_detail::wait_vm_complete();
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t *slot = vshmem_detail::sync_slot(ctx.c, team.start, team.slot);
        vshmem_detail::counter_barrier(ctx.c, slot, (uint64_t)team.size * units_per_pe);
    }
    __syncthreads();
}

__device__ __forceinline__ int shmem_team_sync(const shmem_dctx_t &ctx, const shmemx_dteam_t &team)
{
    vshmem_detail::counter_barrier(ctx.c, vshmem_detail::sync_slot(ctx.c, team.start, team.slot),
                                   (uint64_t)team.size);
    return 0;
}
__device__ __forceinline__ int shmem_team_sync_wave(const shmem_dctx_t &ctx, const shmemx_dteam_t &team)
{
    // One wavefront: its memory counter covers all 64 lanes, so lane 0's
    // release after the wait covers the wave's stores; the acquire runs
    // with every lane active once lane 0 is back.
    vshmem_detail::wait_vm_complete();
    if (__lane_id() == 0)
        vshmem_detail::counter_barrier(ctx.c, vshmem_detail::sync_slot(ctx.c, team.start, team.slot),
                                       (uint64_t)team.size);
    vshmem_detail::acquire_agent();
    return 0;
}
__device__ __forceinline__ int shmem_team_sync_wg(const shmem_dctx_t &ctx, const shmemx_dteam_t &team)
{
    shmemx_team_sync_units(ctx, team, 1);
    return 0;
}

__device__ __forceinline__ shmemx_dteam_t shmemx_team_world(const shmem_dctx_t &ctx)
{
    return shmemx_dteam_t{0, 1, ctx.c.npes, 0};
}
__device__ __forceinline__ void shmem_barrier_all(const shmem_dctx_t &ctx) { shmem_team_sync(ctx, shmemx_team_world(ctx)); }
__device__ __forceinline__ void shmem_barrier_all_wave(const shmem_dctx_t &ctx)
{
    shmem_team_sync_wave(ctx, shmemx_team_world(ctx));
}
__device__ __forceinline__ void shmem_barrier_all_wg(const shmem_dctx_t &ctx)
{
    shmemx_team_sync_units(ctx, shmemx_team_world(ctx), 1);
}

/* ---------------------------------------------------------- collectives */
/* The functions in vshmem_detail move and combine the data; they hold no
 * barrier.  The device collectives below open and close them with one of
 * the team.  A kernel that is one whole collective needs neither: its launch
 * follows, and its end precedes, everything else on its stream. */
namespace vshmem_detail {

constexpr uint64_t kCollChunk = 256ull << 10;   // bytes per task: broadcast, fcollect, alltoall
constexpr uint64_t kRedChunk = 16ull << 10;     // bytes per task: reductions
constexpr int kMcastTile = 16;                  // 16-byte vectors per lane in a multicast tile
constexpr int kRedBatch = 8;                    // member loads in flight per lane before combining

// The work-groups of a collective, numbered across the team: member k's
// work-group `rank` (of nwgs) is worker k * nwgs + rank of size * nwgs.
// (32-bit: a grid has fewer than 2^32 work-groups, and 64-bit division and
// remainder would expand to long vector sequences.)
struct Workers {
    uint32_t w, n;
};
__device__ __forceinline__ Workers team_workers(const shmem_dctx_t &ctx, const shmemx_dteam_t &team, int rank,
                                                int nwgs)
{
    const uint32_t k = (uint32_t)((ctx.me - team.start) / team.stride);
    return Workers{k * (uint32_t)nwgs + (uint32_t)rank, (uint32_t)team.size * (uint32_t)nwgs};
}

// The team barrier that opens a collective; thread 0 computes how the work is
// cut, cut(), between its arrival and its wait, and the others get it through
// LDS: the divisions, four wavefronts of a SIMD taking turns at them, cost a
// broadcast of 64 bytes to 4 members by 1024 threads each 1.2 of its 6.5 us.
template <class F>
__device__ __forceinline__ auto open_collective(const shmem_dctx_t &ctx, const shmemx_dteam_t &team, int nwgs, F cut)
{
    using T = decltype(cut());
    constexpr int N = sizeof(T) / 8;
    static_assert(sizeof(T) == 8 * N, "whole 64-bit words");
    __shared__ uint64_t words[N];
    wait_vm_complete();
    __syncthreads();
    if (threadIdx.x == 0)
        counter_barrier(ctx.c, sync_slot(ctx.c, team.start, team.slot), (uint64_t)team.size * (uint64_t)nwgs, [&] {
            const T m = cut();
            __builtin_memcpy(words, &m, sizeof(T));
        });
    __syncthreads();
    uint64_t u[N];
    T m;
#pragma unroll
    for (int i = 0; i < N; ++i) u[i] = first_lane64(words[i]);
    __builtin_memcpy(&m, u, sizeof(T));
    return m;
}

// Member 0's copy of a symmetric object, and the distance between members.
__device__ __forceinline__ uint8_t *member0(const shmem_dctx_t &ctx, const shmemx_dteam_t &team, const void *sym)
{
    return (uint8_t *)sym + (uint64_t)team.start * ctx.c.stride;
}
__device__ __forceinline__ uint64_t member_stride(const shmem_dctx_t &ctx, const shmemx_dteam_t &team)
{
    return (uint64_t)team.stride * ctx.c.stride;
}

// A multicast of n <= T * blockDim.x vectors, loaded once, then written to
// one member after another, starting at a member that depends on the worker.
// Loads past the end read the last vector again, none under a condition of
// its own (copy_pieces tells why): broadcast of 1 MiB to 64 members, chunks of
// 64 KiB to four of them per task, 17.4 us through the loop of whole tiles
// below, 16.2 so.  For few members, where the loads' latency counts, and for
// small work-groups and tasks, where the loop's sixteen conditions do (64
// members, chunks of 8 KiB by 512 threads 78.6 us, 51.8 so; of 4 KiB by 64
// threads 306 and 139): with 64 members per task and four vectors in each of
// 1024 lanes the loop is the faster one (16 MiB 178 us against 182), with two
// as well (32 KiB from each of 64 work-groups 40 us this way, 34 through it).
template <bool NT, int T>
__device__ __forceinline__ void mcast_small(uint8_t *d0, uint64_t pstride, int P, const uint8_t *s, uint32_t n,
                                            uint32_t worker)
{
    const uint32_t i = threadIdx.x, bd = blockDim.x;
    if (i >= n) return;   // wavefronts without a vector load none
    v4u r[T];
#pragma unroll
    for (int u = 0; u < T; ++u) r[u] = ld_any<true, v4u>(s + 16u * min(i + u * bd, n - 1));
    loads_issued();
    int p = (int)(worker % (uint32_t)P);
    for (int k = 0; k < P; ++k) {
        uint8_t *d = d0 + (uint64_t)p * pstride;
#pragma unroll
        for (int u = 0; u < T; ++u)
            if (i + u * bd < n) st<NT>((v4u *)(d + 16u * (i + u * bd)), r[u]);
        if (++p == P) p = 0;
    }
}

// Copy one source range to the same place on every team member (d0 is
// member 0's copy, members pstride apart).  The range goes through a
// register tile: each lane loads kMcastTile 16-byte vectors once, then the
// whole tile is written to one member after another, starting at a member
// that depends on the worker so that concurrent work-groups spread over
// the members.  Long contiguous writes per member page measured about 10%
// faster on MI355X than writing every vector to all members in turn.
// The vectors are the destination's (the same on every member, the member
// stride being a multiple of 16), the loads take the source as it falls, and
// up to two 16-byte pieces at the edges (or, below 16 bytes, single bytes)
// are dealt to the threads member by member.
template <bool NT>
__device__ __forceinline__ void multicast(uint8_t *d0, uint64_t pstride, int P, const uint8_t *src, uint64_t len,
                                          uint32_t worker)
{
    const uint32_t bd = blockDim.x;
    if (len < 16) {
        for (uint32_t q = threadIdx.x; q < (uint32_t)P * (uint32_t)len; q += bd) {
            const uint32_t p = q / (uint32_t)len, i = q - p * (uint32_t)len;
            d0[p * pstride + i] = src[i];
        }
        return;
    }
    const uint64_t head = (16 - ((uintptr_t)d0 & 15)) & 15, nv = (len - head) / 16;
    const bool tail = ((len - head) & 15) != 0;
    if (head || tail)
        for (uint32_t q = threadIdx.x; q < 2 * (uint32_t)P; q += bd)
            if ((q & 1) ? tail : head != 0) {
                const uint64_t o = (q & 1) ? len - 16 : 0;
                st_any<NT, v4u>(d0 + (q >> 1) * pstride + o, ld_any<true, v4u>(src + o));
            }
    if (nv <= kMcastTile / 4 * bd && (P <= 16 || bd <= 512 || nv <= bd)) {
        if (nv) mcast_small<NT, kMcastTile / 4>(d0 + head, pstride, P, src + head, (uint32_t)nv, worker);
        return;
    }
    for (uint64_t i0 = threadIdx.x; i0 < nv; i0 += (uint64_t)kMcastTile * bd) {
        const uint8_t *s = src + head + 16 * i0;
        v4u r[kMcastTile];
#pragma unroll
        for (int u = 0; u < kMcastTile; ++u)
            if (i0 + u * bd < nv) r[u] = ld_any<true, v4u>(s + 16 * u * bd);
        int p = (int)(worker % (uint32_t)P);
        for (int k = 0; k < P; ++k) {
            v4u *d = (v4u *)(d0 + head + (uint64_t)p * pstride) + i0;
#pragma unroll
            for (int u = 0; u < kMcastTile; ++u)
                if (i0 + u * bd < nv) st<NT>(d + u * bd, r[u]);
            if (++p == P) p = 0;
        }
    }
}

// x / d, in 32 bits when both fit (a 64-bit division is a long sequence).
__host__ __device__ __forceinline__ uint64_t udiv(uint64_t x, uint64_t d)
{
    return ((x | d) >> 32) == 0 ? (uint32_t)x / (uint32_t)d : x / d;
}

// How a multicast of Q source ranges of n bytes to P members is cut into
// tasks: chunks of a range (all of one size, no larger than `chunk`, a
// multiple of 4 KiB where they are long) times groups of members.  With
// enough ranges and chunks of the launch's size a task writes its chunk to
// every member, and the chunks shrink until the last round of tasks is full.
// With less than half a task per worker, chunks are at most 64 KiB (four
// vectors per lane of 1024) and the members are split as well, then the
// chunks down to 16 KiB (one vector per lane): re-reading a chunk for each
// group of members costs little, most of the traffic being the writes, and
// an idle CU costs its share.  One 1024-thread work-group per CU, 64 members:
// a broadcast of 1 MiB took 137 us as four tasks of 256 KiB and takes 15;
// fcollect of 300000 bytes 258 us in two rounds, the second a quarter full,
// and 248 in one.  13 members, 256 MiB: chunks of even size but off the line
// boundaries 1099 us, on them 759.
//
// The launchers compute it on the host: its chain of divisions, and the
// instructions it brings in, cost each launch 1.4 us (one launch after another,
// broadcast of 16 bytes over 4 PEs: 4.9 us, and 3.7 from the host, the rate of
// the launches; of 1 MiB over 64: 16.6 and 14.4).
struct McastSplit {
    uint64_t chunk, nch;     // bytes per chunk, chunks per range
    uint32_t per, groups;    // members per task, member groups
};
__host__ __device__ __forceinline__ uint64_t least(uint64_t a, uint64_t b) { return a < b ? a : b; }
__host__ __device__ __forceinline__ uint64_t most(uint64_t a, uint64_t b) { return a < b ? b : a; }
__host__ __device__ __forceinline__ McastSplit mcast_split(uint64_t n, uint32_t Q, uint32_t P, uint32_t workers, uint64_t chunk)
{
    uint64_t c = chunk, k = udiv(n + c - 1, c);
    if (2 * k * Q < workers) {
        c = least(c, 64u << 10);
        k = udiv(n + c - 1, c);
        for (; c > (16u << 10) && k * Q * P < workers; c >>= 1) k *= 2;
    }
    // Whole rounds: as many groups as leave every task a worker of its own,
    // then as many chunks as fill the last round.
    uint32_t g = 1;
    if (k * Q < workers) {
        g = (uint32_t)least(P, workers / ((uint32_t)k * Q));
        k = most(k, workers / (g * Q));
    } else {
        k = udiv(udiv(k * Q + workers - 1, workers) * workers, Q);
    }
    McastSplit m;
    const uint64_t even = udiv(n + k - 1, k), line = even >= (16u << 10) ? 4096 : 16;
    m.chunk = least((even + line - 1) & ~(line - 1), chunk);
    m.nch = udiv(n + m.chunk - 1, m.chunk);
    m.per = (P + g - 1) / g;
    m.groups = (P + m.per - 1) / m.per;
    return m;
}

// The Q ranges of a broadcast (Q = 1) or fcollect (Q = P): range q is n
// bytes at src + q * sstep and goes to dest + q * n on every member.
// Neighbouring tasks are chunks of one range for one group: the work-groups
// that run together write neighbouring runs of the same members (with the
// groups of one chunk as neighbours, 13 members, 256 MiB: 919 us against
// 742).
template <bool NT>
__device__ __forceinline__ void multicast_all(uint8_t *D, uint64_t ps, uint32_t P, const uint8_t *src, uint64_t sstep,
                                              uint32_t Q, uint64_t n, const Workers &W, const McastSplit &m)
{
    const uint64_t ntask = m.nch * Q * m.groups;
    for (uint64_t t = W.w; t < ntask; t += W.n) {
        const uint64_t r = m.nch == 1 ? t : udiv(t, m.nch), g = Q == 1 ? r : udiv(r, Q), q = r - g * Q;
        const uint64_t off = (t - r * m.nch) * m.chunk;
        const uint32_t p0 = (uint32_t)g * m.per;
        multicast<NT>(D + p0 * ps + q * n + off, ps, (int)min(m.per, P - p0), src + q * sstep + off,
                      min(m.chunk, n - off), W.w);
    }
}

// Member p's block q <- a block of member q, n bytes each: block p of its
// source (alltoall) or its only one (fcollect of small blocks).  Nothing
// here needs a work-group together, so a task is one chunk of one block and
// goes to one wavefront: chunks of whole batches (U 16-byte vectors per
// lane), about eight to a wavefront where the blocks allow it, so that
// wavefronts end together whatever the block size.  Blocks shorter than a
// batch go to a group of g lanes, the smallest power of two that covers one
// in a pass, at most a wavefront and never more than the work-group has.
// Consecutive tasks go to different work-groups first, so a few tiny blocks
// per member still spread over every work-group.
//
// 64 members, one 1024-thread work-group per CU: blocks of 300000 bytes took
// 466 us cut into even chunks per work-group (whose last, partly filled batch
// is a round trip of its own) and take 437, blocks of 100001 bytes 166 and 159,
// 1 MiB 1480 and 1460.  Few wavefronts feel each task: where a wavefront has
// eight blocks or more they stay whole (a task is two more pages to translate:
// 64 members, one wavefront each, 100000 bytes 719 us in two tasks per block,
// 575 in one), and a unit steps from task to task without a division.
struct PairSplit {
    uint64_t task, nch;   // bytes per task, tasks per block
    uint64_t schunk;      // a unit's next task: this many further in its block,
    uint32_t sq, sp;      // source members and destination members
    uint32_t g, pad;      // lanes per task
};
template <int U>
__host__ __device__ __forceinline__ PairSplit pair_split(uint64_t n, uint32_t P, uint32_t workers, uint32_t bd, uint64_t chunk)
{
    constexpr uint64_t kPass = 16ull * U, kBatch = 64 * kPass;   // bytes per lane and per wavefront in one pass
    // (Work-groups below a wavefront count as one.)
    const uint64_t share = udiv(n * P * P, (uint64_t)workers * most(bd / 64, 1) * 8);
    PairSplit m;
    // Split for balance, but where a unit has eight blocks or more; even then
    // in equal tasks, no larger than a chunk.
    const uint64_t parts = udiv(n + chunk - 1, chunk), even = (udiv(n + parts - 1, parts) + kBatch - 1) / kBatch * kBatch;
    m.task = least(least(chunk, n), share >= n ? even : most(kBatch, least(share / kBatch * kBatch, 64u << 10)));
    m.g = bd < 2 ? 1 : 2;
    while (m.g < 64 && 2 * m.g <= bd && m.g * kPass < m.task) m.g <<= 1;
    m.pad = 0;
    m.nch = udiv(n + m.task - 1, m.task);
    const uint64_t step = (uint64_t)workers * (bd / m.g), blocks = udiv(step, m.nch);
    m.schunk = step - blocks * m.nch;
    m.sp = (uint32_t)udiv(blocks, P);
    m.sq = (uint32_t)(blocks - (uint64_t)m.sp * P);
    return m;
}
// Unit `unit` (of W.n * groups) takes tasks unit, unit + W.n * groups, ...
template <bool NT, int U, bool ONE>
__device__ __forceinline__ void pair_tasks(uint8_t *D0, const uint8_t *S0, uint64_t ps, uint32_t P, uint64_t n,
                                           uint64_t unit, uint64_t lane, uint64_t nl, const PairSplit &m)
{
    const uint64_t blk = m.nch == 1 ? unit : udiv(unit, m.nch);
    uint64_t c = unit - blk * m.nch;                       // chunk of the block
    uint64_t p = udiv(blk, P);                             // destination member
    uint32_t q = (uint32_t)(blk - p * P);                  // source member
    while (p < P) {
        const uint64_t off = c * m.task;
        copy_bytes<U, NT>(D0 + p * ps + q * n + off, S0 + q * ps + (ONE ? 0 : p * n) + off, min(m.task, n - off),
                          lane, nl);
        c += m.schunk;
        q += m.sq;
        p += m.sp;
        if (c >= m.nch) {
            c -= m.nch;
            ++q;
        }
        if (q >= P) {
            q -= P;
            ++p;
        }
    }
}
template <bool NT, int U, bool ONE>
__device__ __forceinline__ void pair_blocks(uint8_t *D0, const uint8_t *S0, uint64_t ps, uint32_t P, uint64_t n,
                                            const Workers &W, const PairSplit &m)
{
    const uint32_t g = m.g;
    if (g == 64) {
        // A wavefront's tasks: their places stay in scalar registers.
        const uint32_t mine = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        if ((mine + 1) * 64 <= blockDim.x)
            pair_tasks<NT, U, ONE>(D0, S0, ps, P, n, (uint64_t)mine * W.n + W.w, threadIdx.x & 63, 64, m);
    } else {
        const uint32_t mine = threadIdx.x >> __builtin_ctz(g);
        if ((mine + 1) * g <= blockDim.x)   // not past the last whole group
            pair_tasks<NT, U, ONE>(D0, S0, ps, P, n, (uint64_t)mine * W.n + W.w, threadIdx.x & (g - 1), g, m);
    }
}

// fcollect: blocks shorter than kPairMax go from each source to each
// destination, many at once; longer ones are read once per group of members.
// With fewer than eight wavefronts per member too few loads are in flight, and
// a multicast's stores wait for none: 64 members, one wavefront each, 4 KiB
// 36.2 us as pairs and 11.3; four each, 14.0 and 9.3 (10000 bytes 25.4 and
// 12.8); eight each, 64 bytes 3.7 as pairs (four each, 7.9 as multicasts).
constexpr uint64_t kPairMax = 16ull << 10;
__host__ __device__ __forceinline__ bool use_pairs(uint64_t n, uint32_t P, uint32_t workers, uint32_t bd)
{
    return n < kPairMax && (uint64_t)workers * bd >= 512ull * P;
}

// TREE in streaming form.  Pushing x_0, x_1, ... keeps, for every set bit j
// of the count, the reduction of an aligned block of 2^j consecutive inputs
// (slot j).  Pushing merges equal-sized blocks left to right, which is
// exactly the pairing of one TREE level.  At the end the blocks, largest
// (leftmost) first, are combined right-nested: op(B_a, op(B_b, ... B_z)),
// which is how TREE's carried odd elements meet the full subtrees.
struct OpSum {
    template <typename T> __device__ __forceinline__ static T f(T a, T b) { return a + b; }
};
struct OpMax {
    template <typename T> __device__ __forceinline__ static T f(T a, T b) { return (b > a) ? b : a; }
};

constexpr int kTreeLevels = 9;   // teams of up to 2^9 - 1 members

template <typename A, int E, class OP, int LEVELS = kTreeLevels>
struct TreeAcc {
    A s[LEVELS][E];
    __device__ __forceinline__ void push(uint32_t count, const A (&x)[E])
    {
        // The new input merges with the tz occupied slots below the first
        // free one (tz = trailing ones of count) and lands in slot tz.
        const uint32_t tz = (uint32_t)__builtin_ctz(~count);
        A c[E];
#pragma unroll
        for (int e = 0; e < E; ++e) c[e] = x[e];
#pragma unroll
        for (int j = 0; j < LEVELS; ++j) {
            if ((uint32_t)j < tz) {
#pragma unroll
                for (int e = 0; e < E; ++e) c[e] = OP::f(s[j][e], c[e]);
            } else if ((uint32_t)j == tz) {
#pragma unroll
                for (int e = 0; e < E; ++e) s[j][e] = c[e];
            }
        }
    }
    // count >= 1 inputs pushed.
    __device__ __forceinline__ void result(uint32_t count, A (&r)[E]) const
    {
        bool have = false;
#pragma unroll
        for (int j = 0; j < LEVELS; ++j) {
            if ((count >> j) & 1u) {
                if (!have) {
#pragma unroll
                    for (int e = 0; e < E; ++e) r[e] = s[j][e];
                    have = true;
                } else {
#pragma unroll
                    for (int e = 0; e < E; ++e) r[e] = OP::f(s[j][e], r[e]);
                }
            }
        }
    }
};

// Element codecs: a 16-byte vector of the storage type <-> E accumulators.
struct CodecI64 {
    using A = int64_t;
    static constexpr int E = 2;
    static constexpr int ES = 8;
    __device__ __forceinline__ static void unpack(const v4u &v, A (&x)[E])
    {
        x[0] = (int64_t)(((uint64_t)v.y << 32) | v.x);
        x[1] = (int64_t)(((uint64_t)v.w << 32) | v.z);
    }
    __device__ __forceinline__ static v4u pack(const A (&x)[E])
    {
        v4u v;
        v.x = (uint32_t)x[0];
        v.y = (uint32_t)((uint64_t)x[0] >> 32);
        v.z = (uint32_t)x[1];
        v.w = (uint32_t)((uint64_t)x[1] >> 32);
        return v;
    }
    __device__ __forceinline__ static A load1(const uint8_t *p) { return *(const int64_t *)p; }
    __device__ __forceinline__ static void store1(uint8_t *p, A v) { *(int64_t *)p = v; }
};

struct CodecF32 {
    using A = float;
    static constexpr int E = 4;
    static constexpr int ES = 4;
    __device__ __forceinline__ static void unpack(const v4u &v, A (&x)[E])
    {
        x[0] = __uint_as_float(v.x);
        x[1] = __uint_as_float(v.y);
        x[2] = __uint_as_float(v.z);
        x[3] = __uint_as_float(v.w);
    }
    __device__ __forceinline__ static v4u pack(const A (&x)[E])
    {
        v4u v;
        v.x = __float_as_uint(x[0]);
        v.y = __float_as_uint(x[1]);
        v.z = __float_as_uint(x[2]);
        v.w = __float_as_uint(x[3]);
        return v;
    }
    __device__ __forceinline__ static A load1(const uint8_t *p) { return *(const float *)p; }
    __device__ __forceinline__ static void store1(uint8_t *p, A v) { *(float *)p = v; }
};

// bf16 -> fp32 is exact (the bf16 bits are the high half of the fp32).
// fp32 -> bf16 rounds to nearest, ties to even; NaN stays a quiet NaN.
__device__ __forceinline__ float bf16_up(uint32_t h) { return __uint_as_float(h << 16); }
__device__ __forceinline__ uint32_t bf16_down(float f)
{
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (u >> 16) | 0x40u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

struct CodecBF16 {
    using A = float;
    static constexpr int E = 8;
    static constexpr int ES = 2;
    __device__ __forceinline__ static void unpack(const v4u &v, A (&x)[E])
    {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[2 * i] = bf16_up(w[i] & 0xFFFFu);
            x[2 * i + 1] = bf16_up(w[i] >> 16);
        }
    }
    __device__ __forceinline__ static v4u pack(const A (&x)[E])
    {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = bf16_down(x[2 * i]) | (bf16_down(x[2 * i + 1]) << 16);
        v4u v;
        v.x = w[0];
        v.y = w[1];
        v.z = w[2];
        v.w = w[3];
        return v;
    }
    __device__ __forceinline__ static A load1(const uint8_t *p) { return bf16_up(*(const uint16_t *)p); }
    __device__ __forceinline__ static void store1(uint8_t *p, A v) { *(uint16_t *)p = (uint16_t)bf16_down(v); }
};

// The vectors of a reduction of nelem elements: 16-byte vectors of the
// destination (the same on every member, the member stride being a multiple
// of 16), from element `head` on, `nvec` of them; the elements before and
// after them are taken one by one.  Loads take the source as it falls.  (A
// destination that is no whole number of elements from a boundary has
// unaligned vectors too.)
struct RedRange {
    uint64_t head, nvec;
};
__host__ __device__ __forceinline__ RedRange red_range(const uint8_t *d0, uint64_t nelem, uint32_t ES)
{
    const uint64_t dm = (uintptr_t)d0 & 15;
    const uint64_t head = dm % ES ? 0 : least(((16 - dm) & 15) / ES, nelem);
    return RedRange{head, (nelem - head) * ES / 16};
}

// Elements [0, lo) and [hi, nelem), at most 2 (16 / ES) - 2 of them, one
// wavefront each: lane p loads member p's element (of each 64 members), TREE
// is taken level by level between the lanes, and each lane stores the result
// to its member.  One lane per element walked the members one load after
// another: with 64 members, the three last of 100003 elements took 12 of the
// call's 30 us.  Work-groups that are no whole wavefronts do that still.
// Elements go to different work-groups, the last ones first: those are dealt
// fewer tasks when tasks run out.
template <class CODEC, class OP>
__device__ __forceinline__ void reduce_singles(int P, uint64_t pstride, const uint8_t *s0, uint8_t *d0, uint64_t nelem,
                                               uint64_t lo, uint64_t hi, const Workers &W)
{
    using A = typename CODEC::A;
    const uint64_t nsingle = lo + (nelem - hi);
    if (nsingle == 0) return;
    if (blockDim.x & 63) {
        for (uint64_t q = (uint64_t)W.w * blockDim.x + threadIdx.x; q < nsingle; q += (uint64_t)W.n * blockDim.x) {
            const uint64_t k = q < lo ? q : hi + (q - lo);
            TreeAcc<A, 1, OP> acc;
            for (int p = 0; p < P; ++p) {
                A x[1] = {CODEC::load1(s0 + (uint64_t)p * pstride + k * CODEC::ES)};
                acc.push((uint32_t)p, x);
            }
            A r[1];
            acc.result((uint32_t)P, r);
            for (int p = 0; p < P; ++p) CODEC::store1(d0 + (uint64_t)p * pstride + k * CODEC::ES, r[0]);
        }
        return;
    }
    const uint32_t lane = __lane_id();
    for (uint64_t q = (uint64_t)(threadIdx.x / 64) * W.n + (W.n - 1 - W.w); q < nsingle;
         q += (uint64_t)W.n * (blockDim.x / 64)) {
        const uint64_t k = q < lo ? q : hi + (q - lo);
        TreeAcc<A, 1, OP> acc;   // over the blocks of 64 members
        uint32_t nb = 0;
        for (int p0 = 0; p0 < P; p0 += 64, ++nb) {
            int len = min(P - p0, 64);
            A x[1] = {A(0)};
            if ((int)lane < len) x[0] = CODEC::load1(s0 + (uint64_t)(p0 + (int)lane) * pstride + k * CODEC::ES);
            for (; len > 1; len = (len + 1) / 2) {
                const A a = __shfl(x[0], (int)(2 * lane) & 63, 64), b = __shfl(x[0], (int)(2 * lane + 1) & 63, 64);
                if ((int)(2 * lane + 1) < len) x[0] = OP::f(a, b);
                else if ((int)(2 * lane) < len) x[0] = a;
            }
            x[0] = __shfl(x[0], 0, 64);
            acc.push(nb, x);
        }
        A r[1];
        acc.result(nb, r);
        for (int p = (int)lane; p < P; p += 64) CODEC::store1(d0 + (uint64_t)p * pstride + k * CODEC::ES, r[0]);
    }
}

// Every member's dest[k] <- TREE over members of src[k], for k < nelem.
// Each lane owns K 16-byte vectors of the range, blockDim.x vectors apart:
// it loads them from every member (kRedBatch loads in flight), folds each
// in member order and writes the results to every member.  With K > 1 a
// wavefront's consecutive loads and stores fall K times in a row into one
// member's page, so each address translation serves K KiB instead of 1
// KiB: the member walk visits 2P pages per vector, more than a CU's
// first-level translation cache holds.  LEVELS bounds the team size
// (2^LEVELS - 1 members).
struct RedSplit {
    RedRange range;
    uint64_t vpt, ntask;   // vectors per task, tasks
};
__host__ __device__ __forceinline__ RedSplit red_split(const uint8_t *d0, uint64_t nelem, uint32_t ES, uint32_t workers,
                                                       uint64_t chunk)
{
    // Vectors per task: the chunk, or an even share per worker when that is
    // smaller, so a small reduction still spreads over every work-group
    // (each element's order over the members does not depend on who runs it).
    // Shares are whole 1 KiB runs: tasks that begin off the lines' boundaries
    // write parts of lines (64 members, bf16, 4000003 elements in 512 tasks
    // of 977 vectors 208 us, of 1024 178).
    RedSplit m;
    m.range = red_range(d0, nelem, ES);
    uint64_t share = udiv(m.range.nvec + workers - 1, workers);
    if (share > 64) share = (share + 63) & ~63ull;
    m.vpt = most(1, least(chunk / 16, share));
    m.ntask = udiv(m.range.nvec + m.vpt - 1, m.vpt);
    return m;
}
template <class CODEC, class OP, bool NT, int K = 1, int LEVELS = kTreeLevels>
__device__ __forceinline__ void reduce(uint8_t *d0, const uint8_t *s0, uint64_t pstride, int P, uint64_t nelem,
                                       const Workers &W, const RedSplit &m)
{
    using A = typename CODEC::A;
    constexpr int E = CODEC::E;
    constexpr int B = kRedBatch / K > 0 ? kRedBatch / K : 1;   // members per load batch
    const uint64_t h = m.range.head, nvec = m.range.nvec, vpt = m.vpt, ntask = m.ntask;
    reduce_singles<CODEC, OP>(P, pstride, s0, d0, nelem, h, h + nvec * 16 / CODEC::ES, W);
    const uint8_t *sv = s0 + h * CODEC::ES;
    uint8_t *dv = d0 + h * CODEC::ES;
    const uint64_t bd = blockDim.x;
    for (uint64_t t = W.w; t < ntask; t += W.n) {
        const uint64_t v1 = min(nvec, (t + 1) * vpt);
        for (uint64_t i = t * vpt + threadIdx.x; i < v1; i += K * bd) {
            TreeAcc<A, E, OP, LEVELS> acc[K];
            const uint8_t *sp = sv + i * 16;
            for (int p0 = 0; p0 < P; p0 += B) {
                v4u raw[B][K];
#pragma unroll
                for (int u = 0; u < B; ++u)
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        if (p0 + u < P && i + k * bd < v1)
                            raw[u][k] = ld_any<NT, v4u>(sp + k * bd * 16 + (uint64_t)(p0 + u) * pstride);
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    if (p0 + u < P) {
#pragma unroll
                        for (int k = 0; k < K; ++k) {
                            A x[E];
                            CODEC::unpack(raw[u][k], x);
                            acc[k].push((uint32_t)(p0 + u), x);
                        }
                    }
                }
            }
            v4u out[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                A r[E];
                acc[k].result((uint32_t)P, r);
                out[k] = CODEC::pack(r);
            }
            uint8_t *dp = dv + i * 16;
            for (int p = 0; p < P; ++p, dp += pstride)
#pragma unroll
                for (int k = 0; k < K; ++k)
                    if (i + k * bd < v1) st_any<NT, v4u>(dp + k * bd * 16, out[k]);
        }
    }
}

// Reduce-to-all with the team's members split over the work-group's
// wavefronts.  Member block b is members [8b, 8b + 8) (the last may be
// shorter).  TREE over all members equals TREE over the blocks' TREE
// results: TREE's first three levels pair elements only inside aligned
// blocks of eight, and a block's last element is carried exactly when it
// is the list's last.  Per step, wavefront w folds block b of one tile of
// 64 vectors (one vector per lane, the block's up to 8 loads in flight),
// leaves the block result in LDS, and after one work-group barrier every
// wavefront of the tile folds the tile's block results in block order and
// stores the packed result to its own block's members.  A work-group of
// `waves` wavefronts serves teams of up to 8 * waves members and works on
// waves / m tiles per step (m = number of blocks); its tasks are `chunk`
// bytes of every member, walked tile by tile.  The LDS block results
// are double-buffered, so one barrier per step suffices.  Every thread of
// the work-group calls it; blockDim.x is a multiple of 64, at most
// 64 * kRedWaveMax.
// Bound by latency where it is chosen by itself (a tile or two per
// work-group): a block's loads are under no condition and the fold of the
// block results is unrolled, 64 members, 4096 elements of fp32 6.6 -> 5.1 us.
// (Block and tile in scalar registers take 81 registers instead of 142, but
// 0.7 us more.)
constexpr int kRedWaveMax = 8;

struct RedWavesSplit {
    RedRange range;
    uint64_t tpt, ntask;   // tiles of 64 vectors per task, tasks
    uint32_t m, G;         // member blocks, tiles per step
};
// Bytes per member that a work-group takes in one step.
__host__ __forceinline__ uint64_t red_step_bytes(uint32_t P, uint32_t waves) { return 1024ull * (waves / ((P + 7) / 8)); }
__host__ __forceinline__ RedWavesSplit red_waves_split(const uint8_t *d0, uint64_t nelem, uint32_t ES, uint32_t P,
                                                       uint32_t waves, uint64_t chunk)
{
    RedWavesSplit k;
    k.range = red_range(d0, nelem, ES);
    k.tpt = chunk >= 1024 ? chunk / 1024 : 1;
    k.ntask = ((k.range.nvec + 63) / 64 + k.tpt - 1) / k.tpt;
    k.m = (P + 7) / 8;
    k.G = waves / k.m;
    return k;
}
template <class CODEC, class OP, bool NT>
__device__ __forceinline__ void reduce_waves(uint8_t *d0, const uint8_t *s0, uint64_t pstride, int P, uint64_t nelem,
                                             const Workers &W, const RedWavesSplit &k)
{
    using A = typename CODEC::A;
    constexpr int E = CODEC::E;
    __shared__ A part[2][kRedWaveMax][E][64];
    const uint32_t w = threadIdx.x / 64, lane = __lane_id();
    const uint32_t m = k.m, G = k.G;
    const uint32_t j = w / m, b = w - j * m;           // this wavefront's tile slot and block
    const int p0 = 8 * (int)b, p1 = min(p0 + 8, P);
    const uint64_t h = k.range.head, nvec = k.range.nvec;
    reduce_singles<CODEC, OP>(P, pstride, s0, d0, nelem, h, h + nvec * 16 / CODEC::ES, W);
    const uint8_t *sv = s0 + h * CODEC::ES;
    uint8_t *dv = d0 + h * CODEC::ES;
    // Tasks of `chunk` bytes per member (whole tiles of 64 vectors), dealt to
    // the workers round robin; a worker walks its task's tiles in order.
    const uint64_t ntile = (nvec + 63) / 64, tpt = k.tpt, ntask = k.ntask;
    int buf = 0;
    for (uint64_t task = W.w; task < ntask; task += W.n)
    for (uint64_t t0 = task * tpt; t0 < (task + 1) * tpt && t0 < ntile; t0 += G) {
        const uint64_t i = (t0 + j) * 64 + lane;
        const bool mine = j < G && t0 + j < (task + 1) * tpt && i < nvec;
        if (mine) {
            const uint8_t *sp = sv + i * 16 + (uint64_t)p0 * pstride;
            v4u raw[8];   // (a short block's last member again: no load under a condition of its own)
#pragma unroll
            for (int u = 0; u < 8; ++u) raw[u] = ld_any<NT, v4u>(sp + (uint64_t)min(u, p1 - p0 - 1) * pstride);
            loads_issued();
            TreeAcc<A, E, OP, 4> acc;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (p0 + u < p1) {
                    A x[E];
                    CODEC::unpack(raw[u], x);
                    acc.push((uint32_t)u, x);
                }
            }
            A r[E];
            acc.result((uint32_t)(p1 - p0), r);
#pragma unroll
            for (int e = 0; e < E; ++e) part[buf][w][e][lane] = r[e];
        }
        __syncthreads();
        if (mine) {
            TreeAcc<A, E, OP, 4> acc;
#pragma unroll
            for (uint32_t bb = 0; bb < kRedWaveMax; ++bb) {
                if (bb < m) {
                    A x[E];
#pragma unroll
                    for (int e = 0; e < E; ++e) x[e] = part[buf][j * m + bb][e][lane];
                    acc.push(bb, x);
                }
            }
            A r[E];
            acc.result(m, r);
            const v4u out = CODEC::pack(r);
            uint8_t *dp = dv + i * 16 + (uint64_t)p0 * pstride;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (p0 + u < p1) st_any<NT, v4u>(dp + (uint64_t)u * pstride, out);
        }
        buf ^= 1;
    }
}

} // namespace vshmem_detail

namespace vshmem_detail {
/* Debug check of a collective call: the team lies inside the world and has
 * the caller as a member, both ranges are inside PE 0's user heap, `extra`
 * holds, and the work-group's threads agree on (dest, src, n, tag). */
__device__ __forceinline__ bool coll_ok(const shmem_dctx_t &ctx, const shmemx_dteam_t &team, const void *dest,
                                        uint64_t dbytes, const void *src, uint64_t sbytes, bool extra, uint64_t n,
                                        uint64_t tag)
{
    if (!ctx.c.debug) return true;
    const bool team_ok = team.size >= 1 && team.stride >= 1 && team.start >= 0 &&
                         (int64_t)team.start + (int64_t)(team.size - 1) * team.stride < ctx.c.npes &&
                         ctx.me >= team.start && (ctx.me - team.start) % team.stride == 0 &&
                         (ctx.me - team.start) / team.stride < team.size;
    const bool ok = checked(ctx, team_ok && extra && in_user_heap(ctx, dest, dbytes) && in_user_heap(ctx, src, sbytes));
    return wg_agree(ctx, ok, VSHMEM_U64(dest), VSHMEM_U64(src), n, tag);
}
} // namespace vshmem_detail

/* Team collectives (Section 6.3 names broadcast and reductions among the
 * device-initiated operations; fcollect and alltoall follow OpenSHMEM).
 * Pointers are canonical symmetric addresses; n counts bytes for the
 * data-movement routines and elements for the reductions.
 *
 *   _wg    one work-group per member calls it;
 *   _grid  nwgs work-groups per member call it, this one being `rank`
 *          (0 <= rank < nwgs) among those acting for its PE; the work is
 *          spread over all team.size * nwgs of them.
 *
 * Every participant passes identical arguments (rank aside) and all of them
 * must be resident together.  Each routine starts and ends with a barrier
 * of the team (at its slot), so sources may be rewritten and destinations
 * read, on any member, as soon as it returns.  Destination and source must
 * not overlap (a reduction may run in place).  Reductions fold members in
 * the fixed TREE order (pairs of neighbours, level by level), so results
 * are reproducible bit for bit; bf16 accumulates in fp32 and rounds once to
 * nearest-even; teams of 512 or more members get SHMEMX_ERR_UNSUPPORTED
 * from the reductions, which then do nothing.  With debug checks on, a call
 * whose arguments fail them returns SHMEMX_ERR_ARG before any barrier.
 * Return 0 otherwise. */
__device__ __forceinline__ int shmemx_broadcastmem_grid(const shmem_dctx_t &ctx, const shmemx_dteam_t &team,
                                                        void *dest, const void *src, size_t n, int root, int rank,
                                                        int nwgs)
{
    if (!vshmem_detail::coll_ok(ctx, team, dest, n, src, n, root >= 0 && root < team.size && rank >= 0 && rank < nwgs,
                                n, ((uint64_t)(uint32_t)nwgs << 32) | (uint32_t)root))
        return SHMEMX_ERR_ARG;
    const vshmem_detail::Workers W = vshmem_detail::team_workers(ctx, team, rank, nwgs);
    const uint32_t P = (uint32_t)team.size;
    const vshmem_detail::McastSplit m = vshmem_detail::open_collective(ctx, team, nwgs, [&] {
        return n ? vshmem_detail::mcast_split(n, 1, P, W.n, vshmem_detail::kCollChunk) : vshmem_detail::McastSplit{};
    });
    if (n) {
        const uint64_t ps = vshmem_detail::member_stride(ctx, team);
        vshmem_detail::multicast_all<false>(vshmem_detail::member0(ctx, team, dest), ps, P,
                                            vshmem_detail::member0(ctx, team, src) + (uint64_t)root * ps, 0, 1, n, W,
                                            m);
    }
    shmemx_team_sync_units(ctx, team, (uint64_t)nwgs);
    return 0;
}
__device__ __forceinline__ int shmem_broadcastmem_wg(const shmem_dctx_t &ctx, const shmemx_dteam_t &team, void *dest,
                                                     const void *src, size_t n, int root)
{
    return shmemx_broadcastmem_grid(ctx, team, dest, src, n, root, 0, 1);
}
__device__ __forceinline__ int shmemx_fcollectmem_grid(const shmem_dctx_t &ctx, const shmemx_dteam_t &team,
                                                       void *dest, const void *src, size_t n, int rank, int nwgs)
{
    if (!vshmem_detail::coll_ok(ctx, team, dest, (uint64_t)n * team.size, src, n, rank >= 0 && rank < nwgs, n,
                                (uint64_t)nwgs))
        return SHMEMX_ERR_ARG;
    const vshmem_detail::Workers W = vshmem_detail::team_workers(ctx, team, rank, nwgs);
    const uint32_t P = (uint32_t)team.size;
    const bool pairs = vshmem_detail::use_pairs(n, P, W.n, blockDim.x);
    struct Cut {
        vshmem_detail::McastSplit m;
        vshmem_detail::PairSplit p;
    };
    const Cut cut = vshmem_detail::open_collective(ctx, team, nwgs, [&] {
        Cut c = {};
        if (n && pairs) c.p = vshmem_detail::pair_split<4>(n, P, W.n, blockDim.x, vshmem_detail::kCollChunk);
        else if (n) c.m = vshmem_detail::mcast_split(n, P, P, W.n, vshmem_detail::kCollChunk);
        return c;
    });
    if (n) {
        const uint64_t ps = vshmem_detail::member_stride(ctx, team);
        uint8_t *D = vshmem_detail::member0(ctx, team, dest);
        const uint8_t *S = vshmem_detail::member0(ctx, team, src);
        if (pairs) vshmem_detail::pair_blocks<false, 4, true>(D, S, ps, P, n, W, cut.p);
        else vshmem_detail::multicast_all<false>(D, ps, P, S, ps, P, n, W, cut.m);
    }
    shmemx_team_sync_units(ctx, team, (uint64_t)nwgs);
    return 0;
}
__device__ __forceinline__ int shmem_fcollectmem_wg(const shmem_dctx_t &ctx, const shmemx_dteam_t &team, void *dest,
                                                    const void *src, size_t n)
{
    return shmemx_fcollectmem_grid(ctx, team, dest, src, n, 0, 1);
}
__device__ __forceinline__ int shmemx_alltoallmem_grid(const shmem_dctx_t &ctx, const shmemx_dteam_t &team,
                                                       void *dest, const void *src, size_t n, int rank, int nwgs)
{
    if (!vshmem_detail::coll_ok(ctx, team, dest, (uint64_t)n * team.size, src, (uint64_t)n * team.size,
                                rank >= 0 && rank < nwgs, n, (uint64_t)nwgs))
        return SHMEMX_ERR_ARG;
    const vshmem_detail::Workers W = vshmem_detail::team_workers(ctx, team, rank, nwgs);
    const uint32_t P = (uint32_t)team.size;
    const vshmem_detail::PairSplit m = vshmem_detail::open_collective(ctx, team, nwgs, [&] {
        return n ? vshmem_detail::pair_split<8>(n, P, W.n, blockDim.x, vshmem_detail::kCollChunk)
                 : vshmem_detail::PairSplit{};
    });
    if (n)
        vshmem_detail::pair_blocks<true, 8, false>(
            vshmem_detail::member0(ctx, team, dest), vshmem_detail::member0(ctx, team, src),
            vshmem_detail::member_stride(ctx, team), P, n, W, m);
    shmemx_team_sync_units(ctx, team, (uint64_t)nwgs);
    return 0;
}
__device__ __forceinline__ int shmem_alltoallmem_wg(const shmem_dctx_t &ctx, const shmemx_dteam_t &team, void *dest,
                                                    const void *src, size_t n)
{
    return shmemx_alltoallmem_grid(ctx, team, dest, src, n, 0, 1);
}

#define VSHMEM_DEVICE_REDUCE(PREFIX, NAME, T, CODEC, OP)                                                             \
    __device__ __forceinline__ int PREFIX##NAME##_reduce_grid(const shmem_dctx_t &ctx, const shmemx_dteam_t &team, \
                                                              T *dest, const T *src, size_t nreduce, int rank,     \
                                                              int nwgs)                                            \
    {                                                                                                              \
        if (!vshmem_detail::coll_ok(ctx, team, dest, nreduce * sizeof(T), src, nreduce * sizeof(T),               \
                                    rank >= 0 && rank < nwgs, nreduce, (uint64_t)nwgs))                            \
            return SHMEMX_ERR_ARG;                                                                                 \
        if (team.size >= (1 << vshmem_detail::kTreeLevels)) return SHMEMX_ERR_UNSUPPORTED;                         \
        const vshmem_detail::Workers W = vshmem_detail::team_workers(ctx, team, rank, nwgs);                      \
        uint8_t *D = vshmem_detail::member0(ctx, team, dest);                                                      \
        const vshmem_detail::RedSplit m = vshmem_detail::open_collective(ctx, team, nwgs, [&] {                    \
            return vshmem_detail::red_split(D, nreduce, sizeof(T), W.n, vshmem_detail::kRedChunk);                 \
        });                                                                                                        \
        vshmem_detail::reduce<vshmem_detail::CODEC, vshmem_detail::OP, true>(                                      \
            D, vshmem_detail::member0(ctx, team, src), vshmem_detail::member_stride(ctx, team), team.size, nreduce, \
            W, m);                                                                                                 \
        shmemx_team_sync_units(ctx, team, (uint64_t)nwgs);                                                         \
        return 0;                                                                                                  \
    }
/* The grid forms carry the shmemx_ prefix; the _wg forms are OpenSHMEM names. */
#define VSHMEM_DEVICE_REDUCE_WG(NAME, GRIDNAME, T)                                                                   \
    __device__ __forceinline__ int NAME##_reduce_wg(const shmem_dctx_t &ctx, const shmemx_dteam_t &team, T *dest,  \
                                                    const T *src, size_t nreduce)                                  \
    {                                                                                                              \
        return GRIDNAME##_reduce_grid(ctx, team, dest, src, nreduce, 0, 1);                                        \
    }
VSHMEM_DEVICE_REDUCE(shmemx_, int64_sum, int64_t, CodecI64, OpSum)
VSHMEM_DEVICE_REDUCE(shmemx_, int64_max, int64_t, CodecI64, OpMax)
VSHMEM_DEVICE_REDUCE(shmemx_, float_sum, float, CodecF32, OpSum)
VSHMEM_DEVICE_REDUCE(shmemx_, float_max, float, CodecF32, OpMax)
VSHMEM_DEVICE_REDUCE(shmemx_, bfloat16_sum, uint16_t, CodecBF16, OpSum)   /* bf16 as its bits */
VSHMEM_DEVICE_REDUCE(shmemx_, bfloat16_max, uint16_t, CodecBF16, OpMax)
VSHMEM_DEVICE_REDUCE_WG(shmem_int64_sum, shmemx_int64_sum, int64_t)
VSHMEM_DEVICE_REDUCE_WG(shmem_int64_max, shmemx_int64_max, int64_t)
VSHMEM_DEVICE_REDUCE_WG(shmem_float_sum, shmemx_float_sum, float)
VSHMEM_DEVICE_REDUCE_WG(shmem_float_max, shmemx_float_max, float)
VSHMEM_DEVICE_REDUCE_WG(shmemx_bfloat16_sum, shmemx_bfloat16_sum, uint16_t)
VSHMEM_DEVICE_REDUCE_WG(shmemx_bfloat16_max, shmemx_bfloat16_max, uint16_t)
#undef VSHMEM_DEVICE_REDUCE
#undef VSHMEM_DEVICE_REDUCE_WG

#endif /* VSHMEM_DEVICE_HPP */
