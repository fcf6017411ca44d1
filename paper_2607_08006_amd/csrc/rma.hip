// Device-initiated put/get traffic patterns, the seeded payload fill, and the
// probes that supply measured ceilings (copy bandwidth, atomic rate, launch
// latency, XCD placement).
#include "runtime.hpp"

using namespace vshmem;

namespace {

// Messages m0 .. m1 - 1 (addresses step apart) by nl lanes (whole
// wavefronts), this one `lane`:
// their pieces of sizeof(V) bytes form one index space that the lanes walk,
// U pieces in flight each, so a message of a few pieces leaves no lane idle
// and costs no round trip of its own.  A message's last piece ends at its
// last byte (it may repeat bytes of the one before).  msg >= sizeof(V).
template <typename V, int U, bool NT>
__device__ __forceinline__ void copy_run(uint8_t *D, const uint8_t *S, uint64_t msg, uint64_t sstep, uint64_t dstep,
                                         uint64_t m0, uint64_t m1, uint32_t lane, uint32_t nl)
{
    constexpr uint32_t A = sizeof(V);
    const uint32_t ppm = (uint32_t)((msg + A - 1) / A), last = (uint32_t)msg - A;
    const uint64_t n = (m1 - m0) * ppm;
    // A wavefront's U pieces per lane are one contiguous run of 64 U; the
    // next batch is the unit's U * nl pieces further.  A step of x pieces is
    // x / ppm messages and x % ppm pieces.
    constexpr uint32_t w = 64;
    const uint32_t first = (lane >> 6) * (U * w) + (lane & 63), far = U * nl - (U - 1) * w;
    const uint32_t wj = w / ppm, wr = w % ppm, fj = far / ppm, fr = far % ppm;
    uint32_t r = first % ppm;
    S += (m0 + first / ppm) * sstep;
    D += (m0 + first / ppm) * dstep;
    auto step = [&](uint32_t j, uint32_t q) {
        r += q;
        if (r >= ppm) {
            r -= ppm;
            ++j;
        }
        S += j * sstep;
        D += j * dstep;
    };
    for (uint64_t k = first; k < n; k += (uint64_t)U * nl) {
        V v[U];
        uint8_t *to[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u) step(wj, wr);
            const uint32_t o = min(r * A, last);
            to[u] = D + o;
            if (k + (uint64_t)u * w < n) v[u] = vshmem_detail::ld_any<NT, V>(S + o);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k + (uint64_t)u * w < n) vshmem_detail::st_any<NT, V>(to[u], v[u]);
        step(fj, fr);
    }
}

// Every virtual PE p issues nmsg messages to targets[p] at the given scope,
// then quiets.  Work-group w acts for PE w / wgs_per_pe.  A unit (a
// wavefront at thread and wavefront scope, a work-group, the PE's whole
// share of the grid) takes a run of consecutive messages, all of them
// non-blocking until the quiet:
//   - messages that follow one another without a gap on both sides move as
//     the one range that they are;
//   - otherwise, messages too short to fill one batch of the unit (U 16-byte
//     vectors per lane) are walked together, piece by piece;
//   - longer ones are copied one after another.
// One message at a time costs a round trip to memory per message while most
// lanes idle: with one wavefront per 1 KiB message, 64 PEs x 8192 messages
// took 422 us (2.5 TB/s) and take 198 (5.4); one lane per 64 B message, 64
// PEs x 16384, 49 us (2.7) and 33 (4.1); 1501 B at odd addresses, 64 PEs x
// 4096, 302 us (2.6) and 147 (5.3).  Messages that are whole batches stay
// one at a time, dealt round robin: a wavefront's 4 KiB messages moved at
// 6.0 TB/s so and at 5.8 as one contiguous range per wavefront.  MAXT is the
// largest work-group the instance accepts.
template <int SCOPE, bool IS_PUT, bool NT, int U, int MAXT>
__global__ void __launch_bounds__(MAXT) k_rma_pattern(shmemx_dctx_pub_t c, const int32_t *__restrict__ targets,
                                                      uint64_t src_off, uint64_t dst_off, uint64_t msg, uint64_t nmsg,
                                                      uint64_t sstep, uint64_t dstep, int wgs_per_pe)
{
    const uint32_t pe = blockIdx.x / (uint32_t)wgs_per_pe;
    const uint32_t rank = blockIdx.x - pe * (uint32_t)wgs_per_pe;
    const int tgt = targets[pe];
    if (tgt < 0) return;
    // Source and destination PE of every message of this PE.
    const int spe = IS_PUT ? (int)pe : tgt;
    const int dpe = IS_PUT ? tgt : (int)pe;
    const uint8_t *S = c.base + (uint64_t)spe * c.stride + src_off;
    uint8_t *D = c.base + (uint64_t)dpe * c.stride + dst_off;
    uint32_t unit = 0, units = 1, lane, nl;
    if constexpr (SCOPE <= SHMEMX_SCOPE_WAVE) {
        const uint32_t waves = blockDim.x / 64;
        unit = rank * waves + threadIdx.x / 64;
        units = (uint32_t)wgs_per_pe * waves;
        lane = __lane_id();
        nl = 64;
    } else if constexpr (SCOPE == SHMEMX_SCOPE_WG) {
        unit = rank;
        units = (uint32_t)wgs_per_pe;
        lane = threadIdx.x;
        nl = blockDim.x;
    } else {
        lane = rank * blockDim.x + threadIdx.x;
        nl = (uint32_t)wgs_per_pe * blockDim.x;
    }
    // (Divisions in 32 bits: 64 PEs, 16 messages of 64 bytes at work-group scope
    // 5.4 us with 64-bit ones, 4.3 with these.)
    const uint64_t q = vshmem_detail::udiv(nmsg, units), rem = nmsg - q * units;
    const uint64_t m0 = unit * q + min<uint64_t>(unit, rem), m1 = m0 + q + (unit < rem);
    if (m0 < m1) {
        const uint64_t batch = 16ull * U * nl;
        const bool batches = vshmem_detail::udiv(msg, batch) * batch == msg && (((uintptr_t)D | dstep) & 15) == 0;
        if (sstep == msg && dstep == msg && !batches)
            vshmem_detail::copy_bytes<U, NT, false, 4>(D + m0 * msg, S + m0 * msg, (m1 - m0) * msg, lane, nl);
        else if (msg >= 16 && !batches && msg < min<uint64_t>(8 * batch, 1u << 30))
            copy_run<vshmem_detail::v4u, 4, NT>(D, S, msg, sstep, dstep, m0, m1, lane, nl);
        else if (msg >= 16)
            for (uint64_t j = unit; j < nmsg; j += units)
                vshmem_detail::copy_bytes<U, NT, false, 4>(D + j * dstep, S + j * sstep, msg, lane, nl);
        else if (msg >= 8)
            copy_run<uint64_t, 4, NT>(D, S, msg, sstep, dstep, m0, m1, lane, nl);
        else
            for (uint64_t j = m0 + lane; j < m1; j += nl)
                vshmem_detail::copy_lone<1, NT>(D + j * dstep, S + j * sstep, msg);
    }
    vshmem_detail::release_wg_at_exit();   // quiet
}

template <int SCOPE, bool IS_PUT>
void launch_pattern(int flags, int grid, int wg, hipStream_t s, const shmemx_dctx_pub_t &c, const int32_t *targets,
                    uint64_t so, uint64_t d, uint64_t m, uint64_t n, uint64_t ss, uint64_t ds, int wgs)
{
    const bool nt = (flags & SHMEMX_LAUNCH_NONTEMPORAL) != 0, deep = (flags & SHMEMX_LAUNCH_DEEP) != 0;
#define VSHMEM_PAT_K(NT, U)                                                                                        \
    do {                                                                                                           \
        if (wg <= 256)                                                                                             \
            hipLaunchKernelGGL((k_rma_pattern<SCOPE, IS_PUT, NT, U, 256>), dim3(grid), dim3(wg), 0, s, c, targets, so, \
                               d, m, n, ss, ds, wgs);                                                              \
        else                                                                                                       \
            hipLaunchKernelGGL((k_rma_pattern<SCOPE, IS_PUT, NT, U, 1024>), dim3(grid), dim3(wg), 0, s, c, targets,    \
                               so, d, m, n, ss, ds, wgs);                                                          \
    } while (0)
    if (nt && deep) VSHMEM_PAT_K(true, 8);
    else if (nt) VSHMEM_PAT_K(true, 4);
    else if (deep) VSHMEM_PAT_K(false, 8);
    else VSHMEM_PAT_K(false, 4);
#undef VSHMEM_PAT_K
}

// ---------------------------------------------------------------- fill
__device__ __forceinline__ uint64_t splitmix_at(uint64_t seed, uint64_t i)
{
    uint64_t z = seed + (i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ void k_fill_random(uint8_t *dst, uint64_t nbytes, uint64_t seed, uint64_t word0)
{
    const uint64_t nw = nbytes / 8;
    uint64_t *d = (uint64_t *)dst;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nw; i += (uint64_t)gridDim.x * blockDim.x)
        d[i] = splitmix_at(seed, word0 + i);
    if (blockIdx.x == 0 && threadIdx.x < (nbytes & 7)) {
        uint64_t w = splitmix_at(seed, word0 + nw);
        dst[nw * 8 + threadIdx.x] = (uint8_t)(w >> (8 * threadIdx.x));
    }
}

__global__ void k_fill_typed(uint8_t *dst, uint64_t count, int dtype, uint64_t seed, uint64_t index0)
{
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t x = splitmix_at(seed, index0 + i);
        if (dtype == SHMEMX_DT_INT64) {
            ((uint64_t *)dst)[i] = x;
        } else {
            const float f = (float)((double)(x >> 40) * 0x1.0p-24 * 2.0 - 1.0);
            if (dtype == SHMEMX_DT_FP32) {
                ((float *)dst)[i] = f;
            } else {
                const uint32_t u = __float_as_uint(f);
                ((uint16_t *)dst)[i] = (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
            }
        }
    }
}

// --------------------------------------------------------------- probes
// Achievable-copy probe in the shape that measured fastest on MI355X: each
// work-group streams contiguous chunks of `cv` vectors (dealt round robin),
// nontemporal loads and stores, 8 vectors in flight per lane.
__global__ void __launch_bounds__(1024) k_probe_copy(vshmem_detail::v4u *__restrict__ d,
                                                     const vshmem_detail::v4u *__restrict__ s, uint64_t nv,
                                                     uint64_t cv)
{
    const uint64_t nch = (nv + cv - 1) / cv;
    for (uint64_t c = blockIdx.x; c < nch; c += gridDim.x) {
        const uint64_t b = c * cv;
        const uint64_t n = min(cv, nv - b);
        vshmem_detail::copy_body<vshmem_detail::v4u, 8, true>(d + b, s + b, n, threadIdx.x, blockDim.x);
    }
}

__global__ void k_probe_atomics(uint64_t *table, uint64_t mask, uint64_t nupd, uint64_t seed, uint64_t *acc)
{
    uint64_t x = 0;
    for (uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; u < nupd; u += (uint64_t)gridDim.x * blockDim.x)
        x ^= __hip_atomic_fetch_add(table + (splitmix_at(seed, u) & mask), 1ull, __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_AGENT);
    if (acc && x) __hip_atomic_fetch_xor(acc, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void k_probe_xcd(int32_t *out, int n)
{
    if (threadIdx.x == 0 && (int)blockIdx.x < n) {
        // XCC_ID hardware register (id 20), bits [3:0].
        uint32_t v = __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20);
        out[blockIdx.x] = (int32_t)(v & 0xf);
    }
}

__global__ void k_probe_empty() {}

}  // namespace

extern "C" {

int shmemx_rma_pattern(int op, int scope, const int32_t *targets, uint64_t src_off, uint64_t dst_off,
                       uint64_t msg_bytes, uint64_t nmsg, uint64_t src_step, uint64_t dst_step,
                       const shmemx_launch_t *launch, void *stream)
{
    if (int rc = check_ready()) return rc;
    shmemx_launch_t tmp;
    const shmemx_launch_t &L = launch_or_default(launch, tmp, 4, 256, 0);
    const State &s = st();
    bool ok = (op == SHMEMX_OP_PUT || op == SHMEMX_OP_GET) && scope >= 0 && scope <= SHMEMX_SCOPE_GRID && targets &&
              valid_wg_size(L.wg_size) && L.wgs_per_pe > 0 && (uint64_t)L.wgs_per_pe * s.npes <= (1ull << 31);
    if (ok && nmsg > 0) {
        uint64_t last = nmsg - 1;
        ok = (src_step == 0 || last <= UINT64_MAX / src_step) && (dst_step == 0 || last <= UINT64_MAX / dst_step) &&
             in_user_heap(src_off, last * src_step) && in_user_heap(src_off + last * src_step, msg_bytes) &&
             in_user_heap(dst_off, last * dst_step) && in_user_heap(dst_off + last * dst_step, msg_bytes) &&
             (nmsg == 1 || dst_step >= msg_bytes);
    }
    if (!ok) {
        set_last_error(SHMEMX_ERR_ARG);
        return SHMEMX_ERR_ARG;
    }
    if (nmsg == 0 || msg_bytes == 0) return SHMEMX_OK;
    const int grid = L.wgs_per_pe * s.npes;
    hipStream_t hs = (hipStream_t)stream;
    shmemx_dctx_pub_t c = pub();
#define VSHMEM_PAT(SC)                                                                                        \
    if (op == SHMEMX_OP_PUT)                                                                                  \
        launch_pattern<SC, true>(L.flags, grid, L.wg_size, hs, c, targets, src_off, dst_off, msg_bytes, nmsg, src_step, \
                                 dst_step, L.wgs_per_pe);                                                     \
    else                                                                                                      \
        launch_pattern<SC, false>(L.flags, grid, L.wg_size, hs, c, targets, src_off, dst_off, msg_bytes, nmsg, src_step, \
                                  dst_step, L.wgs_per_pe);
    switch (scope) {
    case SHMEMX_SCOPE_THREAD: VSHMEM_PAT(SHMEMX_SCOPE_THREAD) break;
    case SHMEMX_SCOPE_WAVE: VSHMEM_PAT(SHMEMX_SCOPE_WAVE) break;
    case SHMEMX_SCOPE_WG: VSHMEM_PAT(SHMEMX_SCOPE_WG) break;
    default: VSHMEM_PAT(SHMEMX_SCOPE_GRID) break;
    }
#undef VSHMEM_PAT
    VSHMEM_HIP(hipGetLastError());
    return SHMEMX_OK;
}

int shmemx_fill_random(void *dst, uint64_t nbytes, uint64_t seed, uint64_t word_offset, void *stream)
{
    if (!dst && nbytes) return SHMEMX_ERR_ARG;
    if (nbytes == 0) return SHMEMX_OK;
    uint64_t nw = nbytes / 8 + 1;
    uint64_t grid = (nw + 255) / 256;
    if (grid > 8192) grid = 8192;
    hipLaunchKernelGGL(k_fill_random, dim3((unsigned)grid), dim3(256), 0, (hipStream_t)stream, (uint8_t *)dst, nbytes,
                       seed, word_offset);
    VSHMEM_HIP(hipGetLastError());
    return SHMEMX_OK;
}

int shmemx_fill_typed(void *dst, uint64_t count, int dtype, uint64_t seed, uint64_t index0, void *stream)
{
    const uint64_t es = dtype == SHMEMX_DT_INT64 ? 8 : dtype == SHMEMX_DT_FP32 ? 4 : 2;
    if (dtype < SHMEMX_DT_INT64 || dtype > SHMEMX_DT_BF16 || (!dst && count) || ((uintptr_t)dst % es))
        return SHMEMX_ERR_ARG;
    if (count == 0) return SHMEMX_OK;
    uint64_t grid = (count + 255) / 256;
    if (grid > 16384) grid = 16384;
    hipLaunchKernelGGL(k_fill_typed, dim3((unsigned)grid), dim3(256), 0, (hipStream_t)stream, (uint8_t *)dst, count,
                       dtype, seed, index0);
    VSHMEM_HIP(hipGetLastError());
    return SHMEMX_OK;
}

int shmemx_probe_copy(void *dst, const void *src, uint64_t nbytes, int nwg, int wg_size, void *stream)
{
    if (!dst || !src || (nbytes & 15) || ((uintptr_t)dst & 15) || ((uintptr_t)src & 15) || nwg <= 0 ||
        !valid_wg_size(wg_size))
        return SHMEMX_ERR_ARG;
    hipLaunchKernelGGL(k_probe_copy, dim3(nwg), dim3(wg_size), 0, (hipStream_t)stream, (vshmem_detail::v4u *)dst,
                       (const vshmem_detail::v4u *)src, nbytes / 16, (uint64_t)(16u << 20) / 16);
    VSHMEM_HIP(hipGetLastError());
    return SHMEMX_OK;
}

int shmemx_probe_atomics(uint64_t *table, uint64_t nwords, uint64_t nupdates, uint64_t seed, uint64_t *acc, void *stream)
{
    if (!table || nwords == 0 || (nwords & (nwords - 1))) return SHMEMX_ERR_ARG;
    hipLaunchKernelGGL(k_probe_atomics, dim3(4096), dim3(256), 0, (hipStream_t)stream, table, nwords - 1, nupdates,
                       seed, acc);
    VSHMEM_HIP(hipGetLastError());
    return SHMEMX_OK;
}

int shmemx_probe_xcd(int32_t *out, int nblocks, void *stream)
{
    if (!out || nblocks <= 0) return SHMEMX_ERR_ARG;
    hipLaunchKernelGGL(k_probe_xcd, dim3(nblocks), dim3(64), 0, (hipStream_t)stream, out, nblocks);
    VSHMEM_HIP(hipGetLastError());
    return SHMEMX_OK;
}

int shmemx_probe_empty(void *stream)
{
    hipLaunchKernelGGL(k_probe_empty, dim3(1), dim3(64), 0, (hipStream_t)stream);
    VSHMEM_HIP(hipGetLastError());
    return SHMEMX_OK;
}

}  // extern "C"
