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

// What a collective's kernel gets: member 0's destination and source, the
// distance between members' copies, the work, and how it is cut.
struct Coll {
    uint8_t *D;
    const uint8_t *S;
    uint64_t ps;
    uint64_t n;          // bytes per block (elements for reduce)
    uint32_t P;
};

// The library's launches run the device collectives' bodies, without their
// opening and closing team barriers: nothing inside a collective depends on
// another work-group's stores, the launch follows all earlier work of its
// stream, and its end completes every store.  With them a reduction of 16 fp32
// elements over 64 PEs took 15.6 us, and took 10.6 without.  Work-group b is
// worker b.
__device__ __forceinline__ vshmem_detail::Workers workers() { return vshmem_detail::Workers{blockIdx.x, gridDim.x}; }

// Broadcast (Q = 1, S the root's source) and fcollect of long blocks (Q = P).
template <bool NT>
__global__ void __launch_bounds__(1024) k_multicast(Coll g, uint64_t sstep, uint32_t Q, vshmem_detail::McastSplit m)
{
    vshmem_detail::multicast_all<NT>(g.D, g.ps, g.P, g.S, sstep, Q, g.n, workers(), m);
}

// Alltoall, and fcollect of short blocks (ONE).
template <bool NT, int U, bool ONE>
__global__ void __launch_bounds__(1024) k_pairs(Coll g, vshmem_detail::PairSplit m)
{
    vshmem_detail::pair_blocks<NT, U, ONE>(g.D, g.S, g.ps, g.P, g.n, workers(), m);
}

template <class CODEC, class OP, bool NT>
__global__ void __launch_bounds__(256) k_reduce(Coll g, vshmem_detail::RedSplit m)
{
    vshmem_detail::reduce<CODEC, OP, NT>(g.D, g.S, g.ps, (int)g.P, g.n, workers(), m);
}

// Two vectors per lane and a TREE stack for teams of up to 127 members.
template <class CODEC, class OP, bool NT>
__global__ void __launch_bounds__(256) k_reduce2(Coll g, vshmem_detail::RedSplit m)
{
    vshmem_detail::reduce<CODEC, OP, NT, 2, 7>(g.D, g.S, g.ps, (int)g.P, g.n, workers(), m);
}

template <class CODEC, class OP, bool NT>
__global__ void __launch_bounds__(64 * vshmem_detail::kRedWaveMax) k_reduce_waves(Coll g, vshmem_detail::RedWavesSplit m)
{
    vshmem_detail::reduce_waves<CODEC, OP, NT>(g.D, g.S, g.ps, (int)g.P, g.n, workers(), m);
}

// ------------------------------------------------------------- launching
// Bytes a member writes per automatically added work-group: one pass of 1024
// lanes.  A further work-group costs its dispatch only, now that it is no
// barrier arrival: 64 PEs, alltoall of 4 KiB blocks takes 5.7 us with four
// per member, broadcast of 64 KiB 4.1 (the rate of the launches) with four;
// both had one, between barriers, and took 15.4 and 46.5.
constexpr uint64_t kAutoBytesPerWg = 16ull << 10;

// Wavefronts per CU that a launch of each collective may count on.  The
// launches do not wait for one another, so these are the interface's limits
// on explicit shapes, not the kernels' occupancy: a grid that the device
// collectives could not hold resident is refused in both forms.
constexpr int kWavesBroadcast = 16, kWavesFcollect = 20, kWavesAlltoallDeep = 20, kWavesAlltoall = 32;
constexpr int kWavesReduce = 20, kWavesReduceBf16 = 12, kWavesReduce2 = 16, kWavesReduce2Bf16 = 8;
constexpr int kWavesReduceSplit = 16, kWavesReduceSplitBf16 = 12;

struct Geo {
    shmemx_dctx_pub_t c;
    shmemx_dteam_t team;
    uint64_t dst_off, src_off;
    uint64_t n;          // bytes per block (elements for reduce)
    uint64_t chunk;      // bytes per task
    int wgs_per_pe;

    Coll coll() const
    {
        const uint64_t first = (uint64_t)team.start * c.stride;
        return Coll{c.base + first + dst_off, c.base + first + src_off, (uint64_t)team.stride * c.stride, n,
                    (uint32_t)team.size};
    }
};

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

// Work-groups of a collective's launch, 0 (with the last error set) when it is
// refused.  When the caller left wgs_per_pe at 0, about auto_wgs, a whole
// number per member, and never more than `waves` wavefronts per CU hold.
unsigned team_grid(int waves, Geo &g, int wg, int64_t auto_wgs, int *rc)
{
    const int per_cu = std::max(1, waves * 64 / wg);
    if (g.wgs_per_pe == 0)
        g.wgs_per_pe = (int)std::max<int64_t>(1, std::min<int64_t>(auto_wgs, per_cu * free_cus()) / g.team.size);
    const int grid = g.wgs_per_pe * g.team.size;
    *rc = check_resident(per_cu, grid, wg, "team collective");
    return *rc ? 0 : (unsigned)grid;
}

template <typename K, typename... Args>
int run(K kernel, unsigned grid, int wg, void *stream, Args... args)
{
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(wg), 0, (hipStream_t)stream, args...);
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
    const unsigned grid = team_grid(kWavesBroadcast, g, L.wg_size, movement_wgs(g, n), &rc);
    if (rc || n == 0) return rc;
    Coll k = g.coll();
    k.S += (uint64_t)root * k.ps;
    const vshmem_detail::McastSplit m = vshmem_detail::mcast_split(n, 1, k.P, grid, g.chunk);
    const bool nt = (L.flags & SHMEMX_LAUNCH_NONTEMPORAL) != 0;
    return run(nt ? k_multicast<true> : k_multicast<false>, grid, L.wg_size, stream, k, (uint64_t)0, 1u, m);
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
    const unsigned grid = team_grid(kWavesFcollect, g, L.wg_size, movement_wgs(g, (uint64_t)n * tsize), &rc);
    if (rc || n == 0) return rc;
    const Coll k = g.coll();
    const bool nt = (L.flags & SHMEMX_LAUNCH_NONTEMPORAL) != 0;
    if (vshmem_detail::use_pairs(n, k.P, grid, (uint32_t)L.wg_size)) {
        const vshmem_detail::PairSplit m = vshmem_detail::pair_split<4>(n, k.P, grid, (uint32_t)L.wg_size, g.chunk);
        return run(nt ? k_pairs<true, 4, true> : k_pairs<false, 4, true>, grid, L.wg_size, stream, k, m);
    }
    const vshmem_detail::McastSplit m = vshmem_detail::mcast_split(n, k.P, k.P, grid, g.chunk);
    return run(nt ? k_multicast<true> : k_multicast<false>, grid, L.wg_size, stream, k, k.ps, k.P, m);
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
    const unsigned grid =
        team_grid(deep ? kWavesAlltoallDeep : kWavesAlltoall, g, L.wg_size, movement_wgs(g, (uint64_t)n * tsize), &rc);
    if (rc || n == 0) return rc;
    const Coll k = g.coll();
    const uint32_t bd = (uint32_t)L.wg_size;
    const vshmem_detail::PairSplit m = deep ? vshmem_detail::pair_split<8>(n, k.P, grid, bd, g.chunk)
                                            : vshmem_detail::pair_split<4>(n, k.P, grid, bd, g.chunk);
    if (nt) return run(deep ? k_pairs<true, 8, false> : k_pairs<true, 4, false>, grid, L.wg_size, stream, k, m);
    return run(deep ? k_pairs<false, 8, false> : k_pairs<false, 4, false>, grid, L.wg_size, stream, k, m);
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
    const bool bf = dtype == SHMEMX_DT_BF16;
    const int64_t P = g.team.size, nvec = (int64_t)(nreduce * es / 16);
    // Without a shape from the caller: a reduction with fewer vectors than
    // lanes of a 256-thread work-group per CU leaves lanes idle and is a chain
    // of P / 8 load batches in each of the others.  Splitting the members over
    // wavefronts makes it one batch.  64 members: 8192 vectors of fp32 11.3 ->
    // 5.6 us, of bf16 15.6 -> 6.4; 40960 of fp32 20.0 -> 16.5; 65536 23.0 ->
    // 24.6; 57 members 49152 19.2 -> 20.2, so up to ten sixteenths of the lanes.
    // 40 members (three of eight wavefronts idle): 32768 11.3 -> 8.7, 49152
    // 12.7 -> 14.8; 32 members (two tiles per step) 32768 7.7 -> 6.5, 36864 9.0
    // -> 10.3: half.  24 and 28 members, two tiles per step: 28672 6.5 -> 5.3 and
    // 7.4 -> 5.8 (int64 7.6 -> 5.7), 36864 7.1 -> 8.4 and 8.6 -> 9.6 (int64 from
    // 32768 on), so seven.  17 members: 8192 4.7 and 4.7, bf16 at 16384 5.5 -> 5.8;
    // 13 members 3.8 -> 5.7: not split.
    const int sixteenths = P > 56 ? 10 : P >= 32 ? 8 : P >= 24 ? 7 : 0;
    const int split_cu = (bf ? kWavesReduceSplitBf16 : kWavesReduceSplit) * 64 / 512;
    if (!waves && !two && (!launch || (launch->wgs_per_pe == 0 && launch->wg_size == 0 && launch->chunk_bytes == 0)) &&
        sixteenths && P <= 64 && 16 * nvec <= sixteenths * free_cus() * 256 && split_cu * free_cus() >= P) {
        waves = true;
        L.wg_size = 512;
        // One tile of 64 vectors per work-group while every tile has one, then
        // what a step of the work-group's wavefronts takes (24 members, fp32,
        // 16384 vectors: 6.0 us with one of two tile slots idle, 4.9 so; 1024
        // vectors of 32 members, int64, 5.3 in steps of two, 4.6 in one).
        g.chunk = nvec <= 64 * (free_cus() / P * P) ? 1024 : vshmem_detail::red_step_bytes((uint32_t)P, 8);
    }
    // Work-groups: two per CU, while each still has 128 vectors (64 members,
    // fp32, 2^20 elements: 91.6 us with two per CU, 94.5 with one; 2^22
    // elements 358 and 355, so above 2048 vectors per CU one); split over
    // wavefronts, one per tile step.
    const int64_t step_vecs = 64 * std::max<int64_t>(1, 8 / ((P + 7) / 8));
    const int64_t per_step = waves ? std::max<int64_t>(64, std::min<int64_t>(g.chunk / 16, step_vecs)) : 128;
    const int64_t aw = std::min<int64_t>((nvec <= 2048 * free_cus() ? 2 : 1) * free_cus(), (nvec + per_step * P - 1) / (per_step * P) * P);
    const bool nt = (L.flags & SHMEMX_LAUNCH_NONTEMPORAL) != 0;
    const int per_cu = waves ? (bf ? kWavesReduceSplitBf16 : kWavesReduceSplit)
                       : two ? (bf ? kWavesReduce2Bf16 : kWavesReduce2)
                             : (bf ? kWavesReduceBf16 : kWavesReduce);
    const unsigned grid = team_grid(per_cu, g, L.wg_size, aw, &rc);
    if (rc) return rc;
    const Coll k = g.coll();
    const vshmem_detail::RedSplit m = vshmem_detail::red_split(k.D, nreduce, (uint32_t)es, grid, g.chunk);
    const vshmem_detail::RedWavesSplit mw =
        waves ? vshmem_detail::red_waves_split(k.D, nreduce, (uint32_t)es, k.P, (uint32_t)L.wg_size / 64, g.chunk)
              : vshmem_detail::RedWavesSplit{};
#define VSHMEM_RED_K(K, SPLIT, CODEC)                                                                     \
    do {                                                                                                  \
        if (op == SHMEMX_RED_SUM)                                                                         \
            return run(nt ? K<CODEC, OpSum, true> : K<CODEC, OpSum, false>, grid, L.wg_size, stream, k, SPLIT); \
        return run(nt ? K<CODEC, OpMax, true> : K<CODEC, OpMax, false>, grid, L.wg_size, stream, k, SPLIT); \
    } while (0)
#define VSHMEM_RED(CODEC)                                                                                 \
    if (waves) VSHMEM_RED_K(k_reduce_waves, mw, CODEC);                                                   \
    if (two) VSHMEM_RED_K(k_reduce2, m, CODEC);                                                           \
    VSHMEM_RED_K(k_reduce, m, CODEC);
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
