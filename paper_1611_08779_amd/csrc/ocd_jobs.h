// ocd_jobs.h -- tables of the batched launch, shared by its kernels and the host.
#pragma once

#include "ocd_internal.h"

namespace ocd {

struct JobDesc {
    Params P;
    int L;
    int npl;   // complex entries per lane
    int pad_[2];
};

// A tile: the vectors vbase .. vbase + nvb - 1 of a job; in the Gram form, those of one
// subcarrier, and of the next JOB_GRAM_SUBCARRIERS - 1 as well.
struct TileDesc {
    int vbase;
    int job;
    int nvb;
    int pad_;
};

// The kernels of a batch, each with its own part of the tile table and queue head: the
// residual form, then the Gram form for up to 8, 16 and 32 users.
constexpr int N_JOB_KERNELS = 4;
constexpr int JOB_GRAM_SUBCARRIERS[N_JOB_KERNELS] = {0, 4, 4, 1};

// Launches the Gram form's kernel `which` (1 .. 3) over ntiles tiles: one workgroup per
// tile, or (persistent) as many as fit the device, popping tiles from *next.
hipError_t launch_jobs_gram(int which, bool f16, bool box, const JobDesc *jobs,
                            const TileDesc *tiles, unsigned int *next, int ntiles, int persistent,
                            hipStream_t s);

}  // namespace ocd
