// ocd_jobs_gram.hip -- the batched launch's tiles in the Gram form (ocd_gram.h): 16 symbols
// of four subcarriers (a wave each) or, above 16 users, of one per tile; one kernel per
// user bound, so that jobs with few users keep the registers and occupancy of their own
// tile shape.
#include "ocd_gram.h"
#include "ocd_jobs.h"

namespace ocd {

template <int UP, GramSymbols SY, bool F16, bool BOX>
__device__ __forceinline__ void job_gram_tile(const Params &P, long w, int s0, int ns, double *lds,
                                              GramUser *us)
{
    constexpr int NW = UP == 32 ? 4 : 1;
    gram_dispatch<UP, F16>(P, [&](auto vec, auto half) {
        gram_tile<UP, SY, F16, BOX, vec(), half(), NW>(P, w, s0, ns, lds, us);
    });
}

// A workgroup's next tile comes from the queue (PERSISTENT) or its block index: two kernels,
// as the loop over tiles keeps values of every variant of a tile in registers, and without
// it three workgroups fit a compute unit above 16 users, not two.
template <int UP, bool F16, bool BOX, bool PERSISTENT>
__global__ __launch_bounds__(GRAM_THREADS, PERSISTENT || UP < 32 ? 2 : 3) void k_jobs_gram(
    const JobDesc *__restrict__ jobs, const TileDesc *__restrict__ tiles,
    unsigned int *__restrict__ next, int ntiles)
{
    using M16 = GramLds<UP, SY_16, UP == 32 ? 4 : 1>;
    using M8 = GramLds<UP, SY_8, UP == 32 ? 4 : 1>;
    __shared__ __align__(16) double lds[M16::DOUBLES > M8::DOUBLES ? M16::DOUBLES : M8::DOUBLES];
    __shared__ GramUser us[M16::SG * UP];
    auto run = [&](int ti) {
        const TileDesc td = tiles[ti];
        const Params P = jobs[__builtin_amdgcn_readfirstlane(td.job)].P;
        const int v = __builtin_amdgcn_readfirstlane(td.vbase);
        const int ns = __builtin_amdgcn_readfirstlane(td.nvb);
        const int w = v / P.S, s0 = v - w * P.S;
        if (P.S <= 8) job_gram_tile<UP, SY_8, F16, BOX>(P, w, s0, ns, lds, us);
        else job_gram_tile<UP, SY_16, F16, BOX>(P, w, s0, ns, lds, us);
    };
    if constexpr (PERSISTENT) {
        __shared__ int s_tile;
        if (threadIdx.x == 0) s_tile = (int)atomicAdd(next, 1u);
        __syncthreads();
        int ti = __builtin_amdgcn_readfirstlane(s_tile);
        while (ti < ntiles) {
            // claim the following tile now; its value is published after this tile
            int claimed = ntiles;
            if (threadIdx.x == 0) claimed = (int)atomicAdd(next, 1u);
            run(ti);
            __syncthreads();   // this tile is done with LDS (and with s_tile)
            if (threadIdx.x == 0) s_tile = claimed;
            __syncthreads();
            ti = __builtin_amdgcn_readfirstlane(s_tile);
        }
    } else {
        if ((int)blockIdx.x < ntiles) run(blockIdx.x);
    }
}

template <int UP, bool F16, bool BOX>
static hipError_t launch_jobs_k(const JobDesc *jobs, const TileDesc *tiles, unsigned int *next,
                                int ntiles, int persistent, hipStream_t s)
{
    if (!persistent) {
        const int most = (int)groups_per_launch(1, GRAM_THREADS);
        for (int t0 = 0; t0 < ntiles; t0 += most) {
            const int n = ntiles - t0 < most ? ntiles - t0 : most;
            hipLaunchKernelGGL((k_jobs_gram<UP, F16, BOX, false>), dim3(n), dim3(GRAM_THREADS), 0, s,
                               jobs, tiles + t0, next, n);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    auto fn = k_jobs_gram<UP, F16, BOX, true>;
    int per_cu = 0, grid = ntiles;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, reinterpret_cast<const void *>(fn), GRAM_THREADS, 0);
    if (e != hipSuccess) return e;
    const long fit = (long)per_cu * device_cu_count();
    if (fit >= 1 && fit < grid) grid = (int)fit;
    hipLaunchKernelGGL(fn, dim3(grid), dim3(GRAM_THREADS), 0, s, jobs, tiles, next, ntiles);
    return hipGetLastError();
}

template <int UP>
static hipError_t launch_jobs_u(bool f16, bool box, const JobDesc *jobs, const TileDesc *tiles,
                                unsigned int *next, int ntiles, int persistent, hipStream_t s)
{
    if (f16) return box ? launch_jobs_k<UP, true, true>(jobs, tiles, next, ntiles, persistent, s)
                        : launch_jobs_k<UP, true, false>(jobs, tiles, next, ntiles, persistent, s);
    return box ? launch_jobs_k<UP, false, true>(jobs, tiles, next, ntiles, persistent, s)
               : launch_jobs_k<UP, false, false>(jobs, tiles, next, ntiles, persistent, s);
}

hipError_t launch_jobs_gram(int which, bool f16, bool box, const JobDesc *jobs,
                            const TileDesc *tiles, unsigned int *next, int ntiles, int persistent,
                            hipStream_t s)
{
    switch (which) {
    case 1: return launch_jobs_u<8>(f16, box, jobs, tiles, next, ntiles, persistent, s);
    case 2: return launch_jobs_u<16>(f16, box, jobs, tiles, next, ntiles, persistent, s);
    case 3: return launch_jobs_u<32>(f16, box, jobs, tiles, next, ntiles, persistent, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ocd
