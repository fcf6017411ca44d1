// Host launchers of the team collectives: broadcast, fcollect, alltoall and
// reductions to all (sum, max) over int64, fp32 and bf16 with fp32
// accumulation, in the fixed TREE order.  The kernels call the device
// collectives of vshmem_device.hpp with launch-chosen task sizes and
// store kinds.
#include <algorithm>
#include <cstdio>

#include "runtime.hpp"

using namespace vshmem;

namespace {

using vshmem_detail::CodecBF16;
using vshmem_detail::CodecF32;
using vshmem_detail::CodecI64;
using vshmem_detail::OpMax;
using vshmem_detail::OpSum;

struct Geo {
    shmemx_dctx_pub_t c;
    shmemx_dteam_t team;
    uint64_t dst_off, src_off;
    uint64_t n;          // bytes per block (elements for reduce)
    uint64_t chunk;      // bytes per task
    int wgs_per_pe;
};

// The library's launches run the device collectives' bodies, without their
// opening and closing team barriers: nothing inside a collective depends on
// another work-group's stores, the launch follows all earlier work of its
// stream, and its end completes every store.  With them a reduction of 16 fp32
// elements over 64 PEs took 15.6 us, and takes 10.6 without.  Work-group b acts for team
// member b / wgs_per_pe, as its rank b % wgs_per_pe.
struct Caller {
    shmem_dctx_t ctx;
    void *dst;
    const void *src;
    int rank;
};

__device__ __forceinline__ Caller caller(const Geo &g)
{
    const int k = (int)(blockIdx.x / (unsigned)g.wgs_per_pe);
    return Caller{shmemx_dctx_bind(g.c, shmemx_team_pe(g.team, k)), g.c.base + g.dst_off, g.c.base + g.src_off,
                  (int)(blockIdx.x - (unsigned)k * (unsigned)g.wgs_per_pe)};
}

template <bool NT>
__global__ void __launch_bounds__(1024) k_broadcast(Geo g, int root)
{
    const Caller a = caller(g);
    vshmem_detail::broadcast<NT>(a.ctx, g.team, a.dst, a.src, g.n, root, a.rank, g.wgs_per_pe, g.chunk);
}

template <bool NT>
__global__ void __launch_bounds__(1024) k_fcollect(Geo g)
{
    const Caller a = caller(g);
    vshmem_detail::fcollect<NT>(a.ctx, g.team, a.dst, a.src, g.n, a.rank, g.wgs_per_pe, g.chunk);
}

template <bool NT, int U>
__global__ void __launch_bounds__(1024) k_alltoall(Geo g)
{
    const Caller a = caller(g);
    vshmem_detail::alltoall<NT, U>(a.ctx, g.team, a.dst, a.src, g.n, a.rank, g.wgs_per_pe, g.chunk);
}

template <class CODEC, class OP, bool NT>
__global__ void __launch_bounds__(256) k_reduce(Geo g)
{
    const Caller a = caller(g);
    (void)vshmem_detail::reduce<CODEC, OP, NT>(a.ctx, g.team, a.dst, a.src, g.n, a.rank, g.wgs_per_pe, g.chunk);
}

// Two vectors per lane and a TREE stack for teams of up to 127 members.
template <class CODEC, class OP, bool NT>
__global__ void __launch_bounds__(256) k_reduce2(Geo g)
{
    const Caller a = caller(g);
    (void)vshmem_detail::reduce<CODEC, OP, NT, 2, 7>(a.ctx, g.team, a.dst, a.src, g.n, a.rank, g.wgs_per_pe,
                                                      g.chunk);
}

template <class CODEC, class OP, bool NT>
__global__ void __launch_bounds__(64 * vshmem_detail::kRedWaveMax) k_reduce_waves(Geo g)
{
    const Caller a = caller(g);
    vshmem_detail::reduce_waves<CODEC, OP, NT>(a.ctx, g.team, a.dst, a.src, g.n, a.rank, g.wgs_per_pe, g.chunk);
}

// ------------------------------------------------------------- launching
// Bytes a member writes per automatically added work-group: one pass of 1024
// lanes.  A further work-group costs its dispatch only, now that it is no
// barrier arrival: 64 PEs, alltoall of 4 KiB blocks takes 7.4 us with four
// per member (the rate at which the host launches), broadcast of 64 KiB 7.1
// with four; both had one, between barriers, and took 15.4 and 46.5.
constexpr uint64_t kAutoBytesPerWg = 16ull << 10;

// Wavefronts per CU that a launch of each collective may count on.  The
// launches do not wait for one another, so these are the interface's limits
// on explicit shapes, not the kernels' occupancy: a grid that the device
// collectives could not hold resident is refused in both forms.
constexpr int kWavesBroadcast = 16, kWavesFcollect = 20, kWavesAlltoallDeep = 20, kWavesAlltoall = 32;
constexpr int kWavesReduce = 20, kWavesReduceBf16 = 12, kWavesReduce2 = 16, kWavesReduce2Bf16 = 8;
constexpr int kWavesReduceSplit = 16, kWavesReduceSplitBf16 = 12;

// CUs the progress kernel leaves free.
int64_t free_cus() { return std::max(0, st().num_cus - progress_reserved_cus()); }

// Work-groups over the team of a data-movement collective whose members
// write bytes_per_member each: about one per CU, fewer when that is little.
// In measurements on MI355X, streaming copies reached higher HBM bandwidth
// with one wide work-group per CU than with the grid filled to its occupancy
// limit.
int64_t movement_wgs(const Geo &g, uint64_t bytes_per_member)
{
    const uint64_t by_bytes = (bytes_per_member + kAutoBytesPerWg - 1) / kAutoBytesPerWg;
    return std::min<int64_t>(free_cus(), (int64_t)std::min<uint64_t>(by_bytes, 1u << 20) * g.team.size);
}

// Launch a collective's kernel.  When the caller left wgs_per_pe at 0, with
// about auto_wgs work-groups, a whole number per member, and never more than
// `waves` wavefronts per CU hold.
template <typename K, typename... Args>
int launch_team_kernel(K kernel, int waves, Geo &g, int wg, hipStream_t s, int64_t auto_wgs, Args... args)
{
    const int per_cu = std::max(1, waves * 64 / wg);
    if (g.wgs_per_pe == 0)
        g.wgs_per_pe = (int)std::max<int64_t>(1, std::min<int64_t>(auto_wgs, per_cu * free_cus()) / g.team.size);
    const int grid = g.wgs_per_pe * g.team.size;
    if (int rc = check_resident(per_cu, grid, wg, "team collective")) return rc;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(wg), 0, s, g, args...);
    VSHMEM_HIP(hipGetLastError());
    return SHMEMX_OK;
}

int make_geo(shmem_team_t team, const void *dest, const void *src, uint64_t dst_bytes, uint64_t src_bytes,
             const shmemx_launch_t *launch, int def_wg, Geo &g, shmemx_launch_t &L, uint64_t def_chunk = 256ull << 10,
             int def_flags = 0)
{
    if (int rc = check_ready()) return rc;
    if (team_get(team, &g.team) != SHMEMX_OK) return SHMEMX_ERR_ARG;
    launch_or_default(launch, L, 1, def_wg, def_chunk);
    if (!launch) L.flags = def_flags;
    if (launch && launch->wgs_per_pe < 0) return SHMEMX_ERR_ARG;
    if (!valid_wg_size(L.wg_size) || (L.chunk_bytes & 15) || (int64_t)L.wgs_per_pe * g.team.size > (1 << 24))
        return SHMEMX_ERR_ARG;
    g.dst_off = sym_offset(dest, dst_bytes);
    g.src_off = sym_offset(src, src_bytes);
    if (g.dst_off == UINT64_MAX || g.src_off == UINT64_MAX) return SHMEMX_ERR_ARG;
    g.c = pub();
    g.chunk = L.chunk_bytes;
    g.wgs_per_pe = launch ? launch->wgs_per_pe : 0;   // 0: the launch's own choice
    return SHMEMX_OK;
}

bool overlap(uint64_t a, uint64_t an, uint64_t b, uint64_t bn) { return a < b + bn && b < a + an; }

}  // namespace

extern "C" {

int shmemx_broadcastmem_launch(shmem_team_t team, void *dest, const void *src, size_t n, int root,
                               const shmemx_launch_t *launch, void *stream)
{
    Geo g{};
    shmemx_launch_t L;
    int rc = make_geo(team, dest, src, n, n, launch, 1024, g, L);
    if (!rc && (root < 0 || root >= g.team.size || overlap(g.dst_off, n, g.src_off, n))) rc = SHMEMX_ERR_ARG;
    if (rc) {
        set_last_error(rc);
        return rc;
    }
    g.n = n;
    if (L.flags & SHMEMX_LAUNCH_NONTEMPORAL)
        return launch_team_kernel(k_broadcast<true>, kWavesBroadcast, g, L.wg_size, (hipStream_t)stream, movement_wgs(g, n), root);
    return launch_team_kernel(k_broadcast<false>, kWavesBroadcast, g, L.wg_size, (hipStream_t)stream, movement_wgs(g, n), root);
}

int shmemx_fcollectmem_launch(shmem_team_t team, void *dest, const void *src, size_t n, const shmemx_launch_t *launch,
                              void *stream)
{
    Geo g{};
    shmemx_launch_t L;
    int rc = SHMEMX_OK;
    if (int r0 = check_ready()) return r0;
    int tsize = shmem_team_n_pes(team);
    if (tsize <= 0) rc = SHMEMX_ERR_ARG;
    if (!rc) rc = make_geo(team, dest, src, (uint64_t)n * tsize, n, launch, 1024, g, L);
    if (!rc && overlap(g.dst_off, (uint64_t)n * tsize, g.src_off, n)) rc = SHMEMX_ERR_ARG;
    if (rc) {
        set_last_error(rc);
        return rc;
    }
    g.n = n;
    if (L.flags & SHMEMX_LAUNCH_NONTEMPORAL)
        return launch_team_kernel(k_fcollect<true>, kWavesFcollect, g, L.wg_size, (hipStream_t)stream, movement_wgs(g, (uint64_t)n * tsize));
    return launch_team_kernel(k_fcollect<false>, kWavesFcollect, g, L.wg_size, (hipStream_t)stream, movement_wgs(g, (uint64_t)n * tsize));
}

int shmemx_alltoallmem_launch(shmem_team_t team, void *dest, const void *src, size_t n, const shmemx_launch_t *launch,
                              void *stream)
{
    Geo g{};
    shmemx_launch_t L;
    if (int r0 = check_ready()) return r0;
    int tsize = shmem_team_n_pes(team);
    int rc = tsize <= 0 ? SHMEMX_ERR_ARG : SHMEMX_OK;
    if (!rc)
        rc = make_geo(team, dest, src, (uint64_t)n * tsize, (uint64_t)n * tsize, launch, 1024, g, L, 256ull << 10,
                      SHMEMX_LAUNCH_NONTEMPORAL | SHMEMX_LAUNCH_DEEP);
    if (!rc && overlap(g.dst_off, (uint64_t)n * tsize, g.src_off, (uint64_t)n * tsize)) rc = SHMEMX_ERR_ARG;
    if (rc) {
        set_last_error(rc);
        return rc;
    }
    g.n = n;
    const bool nt = (L.flags & SHMEMX_LAUNCH_NONTEMPORAL) != 0, deep = (L.flags & SHMEMX_LAUNCH_DEEP) != 0;
    hipStream_t hs = (hipStream_t)stream;
    const int64_t aw = movement_wgs(g, (uint64_t)n * tsize);
    if (nt && deep) return launch_team_kernel(k_alltoall<true, 8>, kWavesAlltoallDeep, g, L.wg_size, hs, aw);
    if (nt) return launch_team_kernel(k_alltoall<true, 4>, kWavesAlltoall, g, L.wg_size, hs, aw);
    if (deep) return launch_team_kernel(k_alltoall<false, 8>, kWavesAlltoallDeep, g, L.wg_size, hs, aw);
    return launch_team_kernel(k_alltoall<false, 4>, kWavesAlltoall, g, L.wg_size, hs, aw);
}

int shmemx_reduce_launch(shmem_team_t team, int dtype, int op, void *dest, const void *src, size_t nreduce,
                         const shmemx_launch_t *launch, void *stream)
{
    Geo g{};
    shmemx_launch_t L;
    const uint64_t es = dtype == SHMEMX_DT_INT64 ? 8 : dtype == SHMEMX_DT_FP32 ? 4 : 2;
    int rc = (dtype < SHMEMX_DT_INT64 || dtype > SHMEMX_DT_BF16 || op < SHMEMX_RED_SUM || op > SHMEMX_RED_MAX)
                 ? SHMEMX_ERR_ARG
                 : SHMEMX_OK;
    // Work-groups of up to 256 threads: one lane folds every member
    // (k_reduce).  Larger ones (up to 512): the members are split over the
    // wavefronts (k_reduce_waves), for teams of at most 8 members per
    // wavefront.
    shmemx_launch_t L0 = launch ? *launch : shmemx_launch_t{0, 256, 16ull << 10, SHMEMX_LAUNCH_NONTEMPORAL, 0};
    if (L0.wg_size == 0) L0.wg_size = 256;
    if (!rc) rc = make_geo(team, dest, src, nreduce * es, nreduce * es, &L0, 256, g, L);
    // In place is allowed; partial overlap is not.
    if (!rc && g.dst_off != g.src_off && overlap(g.dst_off, nreduce * es, g.src_off, nreduce * es)) rc = SHMEMX_ERR_ARG;
    bool waves = L.wg_size > 256;
    // SHMEMX_LAUNCH_DEEP: two vectors per lane (teams of up to 127 members).
    const bool two = !waves && (L.flags & SHMEMX_LAUNCH_DEEP) && g.team.size < 128;
    if (!rc && (L.wg_size > 64 * vshmem_detail::kRedWaveMax || L.chunk_bytes == 0 ||
                (waves && g.team.size > 8 * (L.wg_size / 64))))
        rc = SHMEMX_ERR_ARG;
    if (!rc && g.team.size > 511) rc = SHMEMX_ERR_UNSUPPORTED;   // TreeAcc holds 9 levels
    if (rc) {
        set_last_error(rc);
        return rc;
    }
    g.n = nreduce;
    hipStream_t s = (hipStream_t)stream;
    const bool bf = dtype == SHMEMX_DT_BF16;
    const int64_t P = g.team.size, nvec = (int64_t)(nreduce * es / 16);
    // Without a shape from the caller: a reduction with fewer vectors than
    // half the lanes of a 256-thread work-group per CU leaves lanes idle and
    // is a chain of P / 8 load batches in each of the others.  Splitting the
    // members over wavefronts makes it one batch: 64 members, fp32, 16384
    // vectors 13.2 -> 9.6 us, bf16, 8192 vectors 16.3 -> 8.5, 16 elements
    // 10.7 -> 7.6 (the launch); at 65536 vectors the split form is the slower
    // one (37 us against 25), and so it is for 13 members, two batches (9.8
    // against 7.7 at 16384 vectors).
    const int split_cu = (bf ? kWavesReduceSplitBf16 : kWavesReduceSplit) * 64 / 512;
    if (!waves && !two && (!launch || (launch->wgs_per_pe == 0 && launch->wg_size == 0 && launch->chunk_bytes == 0)) &&
        P >= 32 && P <= 64 && 2 * nvec <= free_cus() * 256 && split_cu * free_cus() >= P) {
        waves = true;
        L.wg_size = 512;
        g.chunk = 1024;   // one tile of 64 vectors
    }
    // Work-groups: two per CU, while each still has 128 vectors (64 members,
    // fp32, 2^20 elements: 91.6 us with two per CU, 94.5 with one; 2^22
    // elements 358 and 355, so above 2048 vectors per CU one); split over
    // wavefronts, one per tile step.
    const int64_t per_step = waves ? 64 * std::max<int64_t>(1, 8 / ((P + 7) / 8)) : 128;
    const int64_t aw = std::min<int64_t>((nvec <= 2048 * free_cus() ? 2 : 1) * free_cus(), (nvec + per_step * P - 1) / (per_step * P) * P);
    const bool nt = (L.flags & SHMEMX_LAUNCH_NONTEMPORAL) != 0;
#define VSHMEM_RED_K(K, W, CODEC)                                                                           \
    do {                                                                                                    \
        const int w_ = bf ? W##Bf16 : W;                                                                    \
        if (op == SHMEMX_RED_SUM)                                                                           \
            return nt ? launch_team_kernel(K<CODEC, OpSum, true>, w_, g, L.wg_size, s, aw)              \
                      : launch_team_kernel(K<CODEC, OpSum, false>, w_, g, L.wg_size, s, aw);            \
        return nt ? launch_team_kernel(K<CODEC, OpMax, true>, w_, g, L.wg_size, s, aw)                  \
                  : launch_team_kernel(K<CODEC, OpMax, false>, w_, g, L.wg_size, s, aw);                \
    } while (0)
#define VSHMEM_RED(CODEC)                                                                                   \
    if (waves) VSHMEM_RED_K(k_reduce_waves, kWavesReduceSplit, CODEC);                                      \
    if (two) VSHMEM_RED_K(k_reduce2, kWavesReduce2, CODEC);                                                 \
    VSHMEM_RED_K(k_reduce, kWavesReduce, CODEC);
    if (dtype == SHMEMX_DT_INT64) {
        VSHMEM_RED(CodecI64)
    } else if (dtype == SHMEMX_DT_FP32) {
        VSHMEM_RED(CodecF32)
    } else {
        VSHMEM_RED(CodecBF16)
    }
#undef VSHMEM_RED
#undef VSHMEM_RED_K
}

}  // extern "C"
