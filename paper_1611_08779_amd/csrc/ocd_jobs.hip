// ocd_jobs.hip -- uneven detection jobs in one persistent launch.
//
// Every job is cut into tiles of consecutive (subcarrier, symbol) vectors.  A
// tile runs exactly the one-problem code: gram_tile for a job in the Gram form (whole
// subcarriers and 16 symbols, ocd_jobs_gram.hip, a kernel per user bound), else
// forward_tile.  The lanes per vector follow from the complex entries each lane holds (NPL): a job with B antennas
// uses L = B / NPL lanes (4, 8, 16 or 32).  The batch tuner picks one of three
// lane modes for the whole batch: NPL = 8 for every job; NPL = 16 for jobs with
// B >= 256 (half the lanes per vector: no reduction across DPP rows) and 8 for
// the others; or in addition NPL = 4 for jobs with B <= 128 (more, shorter lane
// groups).  Exactly 8 users (16 with 4 entries per lane) take the unrolled user
// loop, other multiples of 8 users (at most 8 entries per lane) its chunked form.
// A tile of whole
// subcarriers fills most of a 512-lane workgroup whatever B is, while its H_w
// slots stay within one LDS budget (two tiles per CU).  Tiles are sorted
// longest-first (LPT) and persistent workgroups pop them from a device counter
// until the queue is empty.  The queue reset and the persistent kernel can be
// captured once into a hipGraph and replayed; the job and tile tables live in
// the caller's workspace and are re-uploaded on every call, so the graph never
// holds a job pointer.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "ocd_api_internal.h"
#include "ocd_jobs.h"
#include "ocd_tile.h"

namespace ocd {

constexpr int JOB_THREADS = 512;

// Lane modes of the batch tuner: the complex entries per lane for a job with B
// antennas (the lanes per vector are then B / NPL, rounded up to a power of two).
constexpr int N_LANE_MODES = 3;

static int lane_mode_npl(int mode, int B)
{
    if (mode >= 1 && B > 128) return 16;
    if (mode == 2 && B > 32) return 4;
    return 8;
}

constexpr size_t HEADER_BYTES = 256;

// Two schedules over the same LPT-ordered tile table, in one launch:
//   persistent = 0: one workgroup per tile (grid = number of tiles, tile =
//                   blockIdx.x); the hardware dispatcher starts workgroups as
//                   others retire, so one tile's loads overlap another's work.
//   persistent = 1: a fixed grid; each workgroup claims its next tile from the
//                   queue head while it works on the current one.  Every
//                   workgroup stops when the queue is exhausted.
template <int L, int NPL, int UC, bool F16, bool BOX, bool CHUNKED = false>
__device__ __forceinline__ void job_tile(const Params &P, unsigned char *smem, const Tile &t)
{
    forward_tile<L, NPL, F16, BOX, UC, false, false, CHUNKED>(
        P, carve(smem, P, JOB_THREADS / L, false), t);
}

template <bool F16, bool BOX>
__global__ __launch_bounds__(JOB_THREADS, 4) void k_jobs(const JobDesc *__restrict__ jobs,
                                                      const TileDesc *__restrict__ tiles,
                                                      unsigned int *__restrict__ next, int ntiles,
                                                      int persistent)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_tile;
    int ti = blockIdx.x;
    if (persistent) {
        if (threadIdx.x == 0) s_tile = (int)atomicAdd(next, 1u);
        __syncthreads();
        ti = __builtin_amdgcn_readfirstlane(s_tile);
    }
    while (ti < ntiles) {
        // claim the following tile now; its value is published after this tile
        int claimed = ntiles;
        if (persistent && threadIdx.x == 0) claimed = (int)atomicAdd(next, 1u);
        // the tile and its job are the same for the whole workgroup: keep them in
        // scalar registers (the descriptor is then read with scalar loads)
        const TileDesc td = tiles[ti];
        const int job = __builtin_amdgcn_readfirstlane(td.job);
        const JobDesc &jd = jobs[job];
        const Params P = jd.P;
        Tile t;
        t.vbase = __builtin_amdgcn_readfirstlane(td.vbase);
        t.nvb = __builtin_amdgcn_readfirstlane(td.nvb);
        t.w_first = t.vbase / P.S;
        t.nslots = (t.vbase + t.nvb - 1) / P.S - t.w_first + 1;
        // the unrolled user loop for U = 8 (and U = 16 with 4 entries per lane: with 8,
        // its registers would not fit the budget of four 512-thread workgroups per CU),
        // its chunked form (code 1) for the other multiples of 8 users;
        // plan_jobs builds only the (L, NPL) pairs below (job_shape_built)
        const int npl = jd.npl;
        const int uc = (P.U == 8 && npl <= 8) || (P.U == 16 && npl == 4) ? P.U
                       : (P.U % 8 == 0 && npl <= 8) ? 1 : 0;
        switch (jd.L * 10000 + npl * 100 + uc) {
        case 40800: job_tile<4, 8, 0, F16, BOX>(P, smem, t); break;
        case 40808: job_tile<4, 8, 8, F16, BOX>(P, smem, t); break;
        case 80800: job_tile<8, 8, 0, F16, BOX>(P, smem, t); break;
        case 80808: job_tile<8, 8, 8, F16, BOX>(P, smem, t); break;
        case 160800: job_tile<16, 8, 0, F16, BOX>(P, smem, t); break;
        case 160808: job_tile<16, 8, 8, F16, BOX>(P, smem, t); break;
        case 320800: job_tile<32, 8, 0, F16, BOX>(P, smem, t); break;
        case 320808: job_tile<32, 8, 8, F16, BOX>(P, smem, t); break;
        case 160400: job_tile<16, 4, 0, F16, BOX>(P, smem, t); break;
        case 160408: job_tile<16, 4, 8, F16, BOX>(P, smem, t); break;
        case 160416: job_tile<16, 4, 16, F16, BOX>(P, smem, t); break;
        case 320400: job_tile<32, 4, 0, F16, BOX>(P, smem, t); break;
        case 320408: job_tile<32, 4, 8, F16, BOX>(P, smem, t); break;
        case 320416: job_tile<32, 4, 16, F16, BOX>(P, smem, t); break;
        case 161600: job_tile<16, 16, 0, F16, BOX>(P, smem, t); break;
        case 321600: job_tile<32, 16, 0, F16, BOX>(P, smem, t); break;
        case 40801: job_tile<4, 8, 8, F16, BOX, true>(P, smem, t); break;
        case 80801: job_tile<8, 8, 8, F16, BOX, true>(P, smem, t); break;
        case 160801: job_tile<16, 8, 8, F16, BOX, true>(P, smem, t); break;
        case 320801: job_tile<32, 8, 8, F16, BOX, true>(P, smem, t); break;
        case 160401: job_tile<16, 4, 8, F16, BOX, true>(P, smem, t); break;
        case 320401: job_tile<32, 4, 8, F16, BOX, true>(P, smem, t); break;
        default: break;   // not built: plan_jobs never produces such a job
        }
        if (!persistent) break;
        __syncthreads();   // this tile is done with LDS (and with s_tile)
        if (threadIdx.x == 0) s_tile = claimed;
        __syncthreads();
        ti = __builtin_amdgcn_readfirstlane(s_tile);
    }
}

__global__ void k_reset_queue(unsigned int *next)
{
    if (threadIdx.x < N_JOB_KERNELS) next[threadIdx.x] = 0u;
}

// ------------------------------------------------------------------ host planning

// The tiles of a batch: kernel k's are first[k] .. first[k + 1] - 1, longest first.
struct TileTable {
    std::vector<TileDesc> tiles;
    int first[N_JOB_KERNELS + 1] = {};
};

struct JobsPlan {
    std::vector<JobDesc> jobs;
    // shared and cached per (job shapes, policy), since building and sorting the tiles
    // costs far more host time than a launch
    std::shared_ptr<const TileTable> tiles;
    size_t lds_max = 0;
    bool f16 = false, box = false;
};

static std::mutex g_tiles_mu;
static std::map<std::string, std::shared_ptr<const TileTable>> g_tiles;
static std::string jobs_hash(const ocd_problem *jobs, int n);

// Tile-size policies the batch tuner chooses from:
//   0  every lane group of the workgroup busy (tiles of 512/L vectors)
//   1  tiles of whole subcarriers (a multiple of S vectors), else policy 0
//   2  half-size tiles (more tiles, better balance, less LDS per tile)
constexpr int N_POLICIES = 3;

static int tile_vectors(int policy, int L, int S)
{
    const int cap = JOB_THREADS / L;
    if (policy == 1 && S <= cap) return (cap / S) * S;
    if (policy == 2) return std::max(1, cap / 2);
    return cap;
}

// The (L, NPL) pairs k_jobs is built for (NPL = 4 and 16 only with a run-time U).
static bool job_shape_built(int L, int npl)
{
    if (npl == 8) return L == 4 || L == 8 || L == 16 || L == 32;
    return (npl == 16 || npl == 4) && (L == 16 || L == 32);
}

// The kernel that runs a job (see N_JOB_KERNELS).
static int job_kernel(const Params &P)
{
    if (!gram_form(P.B, P.U, P.W, P.S, P.K)) return 0;
    return P.U <= 8 ? 1 : P.U <= 16 ? 2 : 3;
}

static ocd_status plan_jobs(const ocd_problem *jobs, int n, int policy, int lane_mode,
                            JobsPlan &out)
{
    out = JobsPlan();
    if (n < 1 || !jobs) return OCD_EINVAL;
    out.f16 = jobs[0].storage == OCD_STORE_F16;
    out.box = jobs[0].mode != OCD_MMSE;
    for (int j = 0; j < n; ++j) {
        const ocd_problem *pb = &jobs[j];
        ocd_status st = validate(pb);
        if (st != OCD_OK) return st;
        if ((pb->storage == OCD_STORE_F16) != out.f16) return OCD_EINVAL;
        if ((pb->mode != OCD_MMSE) != out.box) return OCD_EINVAL;
        if (pb->B > 8 * 32) return OCD_EUNSUPPORTED;
        int npl_t = lane_mode_npl(lane_mode, pb->B);
        int L = 4;
        while (npl_t * L < pb->B) L *= 2;
        if (!job_shape_built(L, npl_t)) {   // this job keeps 8 entries per lane
            npl_t = 8;
            L = 4;
            while (npl_t * L < pb->B) L *= 2;
        }
        ocd_plan pl = {L, tile_vectors(policy, L, pb->S), 0, 0};
        Params P;
        int npl, threads;
        size_t lds;
        bool ok = false;
        // keep two tiles per CU: at most half of the LDS (whole subcarriers first)
        const size_t budget = (size_t)lds_limit_bytes() / 2 - 64;
        while (pl.vectors_per_block >= 1) {
            // a job with B <= 16 would take fewer than 8 entries per lane even at 4
            // lanes; it runs at the built width of 8, zero-padded
            if (make_params(pb, pl, nullptr, false, P, npl, threads, lds, npl_t) && npl == npl_t &&
                lds_bytes(P, JOB_THREADS / L, false) <= budget) {
                lds = lds_bytes(P, JOB_THREADS / L, false);
                ok = true;
                break;
            }
            const int v = pl.vectors_per_block;
            pl.vectors_per_block = (v > pb->S && v % pb->S == 0) ? v - pb->S : v / 2;
        }
        if (!ok) return OCD_EUNSUPPORTED;
        JobDesc jd;
        std::memset(&jd, 0, sizeof jd);
        jd.P = P;
        jd.L = L;
        jd.npl = npl_t;
        out.jobs.push_back(jd);
        if (job_kernel(P) == 0) out.lds_max = std::max(out.lds_max, lds);
    }
    char pk[32];
    std::snprintf(pk, sizeof pk, "|p%d|m%d", policy, lane_mode);
    const std::string key = jobs_hash(jobs, n) + pk;
    std::lock_guard<std::mutex> lk(g_tiles_mu);
    auto it = g_tiles.find(key);
    if (it != g_tiles.end()) {
        out.tiles = it->second;
        return OCD_OK;
    }
    auto table = std::make_shared<TileTable>();
    // longest processing time first: cost ~ vectors x sweeps x users x padded antennas,
    // in the Gram form ~ users^2 x antennas + vectors x users x (antennas + sweeps x users)
    struct Costed {
        TileDesc t;
        double cost;
    };
    std::vector<Costed> list;
    for (int k = 0; k < N_JOB_KERNELS; ++k) {
        list.clear();
        for (int j = 0; j < n; ++j) {
            const Params &P = out.jobs[j].P;
            if (job_kernel(P) != k) continue;
            const long nvec = (long)P.W * P.S;
            auto add = [&](long v, long nvb, double cost) {
                list.push_back({{(int)v, j, (int)nvb, 0}, cost});
            };
            if (k == 0) {
                for (long v = 0; v < nvec; v += P.vpb) {
                    const long nvb = std::min<long>(P.vpb, nvec - v);
                    add(v, nvb, (double)nvb * P.K * P.U * P.Bpad);
                }
            } else {
                for (long w = 0; w < P.W; w += JOB_GRAM_SUBCARRIERS[k])
                    for (int s = 0; s < P.S; s += 16) {
                        const int ns = std::min(16, P.S - s);
                        add(w * P.S + s, ns,
                            0.5 * P.U * P.U * P.B + (double)ns * P.U * (P.B + (double)P.K * P.U));
                    }
            }
        }
        std::stable_sort(list.begin(), list.end(),
                         [](const Costed &a, const Costed &b) { return a.cost > b.cost; });
        for (const Costed &c : list) table->tiles.push_back(c.t);
        table->first[k + 1] = (int)table->tiles.size();
    }
    const std::shared_ptr<const TileTable> tiles = table;
    out.tiles = tiles;
    g_tiles[key] = tiles;
    return OCD_OK;
}

static size_t table_bytes(const JobsPlan &jp)
{
    return jp.jobs.size() * sizeof(JobDesc) + jp.tiles->tiles.size() * sizeof(TileDesc);
}

// ------------------------------------------------------------------ launch state

struct Staging {
    void *pinned = nullptr;
    size_t bytes = 0;
    hipEvent_t uploaded = nullptr;
    std::vector<unsigned char> last_jobs;           // job table last uploaded here
    std::shared_ptr<const TileTable> last_tiles;   // tile table last uploaded here
};

struct GraphEntry {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

static std::mutex g_mu;
static std::map<void *, Staging> g_staging;
static std::map<std::string, GraphEntry> g_graphs;
static std::map<std::string, int> g_choice;
static hipStream_t g_capture_stream = nullptr;

// A schedule choice: persistent (1) or one workgroup per tile (0), times a tile
// policy, times a lane mode.
constexpr int N_CHOICES = 2 * N_POLICIES * N_LANE_MODES;
constexpr int DEFAULT_CHOICE = 1;   // one workgroup per tile, whole-subcarrier tiles, NPL 8
static int choice_lane_mode(int c) { return c / (2 * N_POLICIES); }
static int choice_persistent(int c) { return (c / N_POLICIES) % 2; }
static int choice_policy(int c) { return c % N_POLICIES; }
static int make_choice(int lane_mode, int persistent, int policy)
{
    return (lane_mode * 2 + persistent) * N_POLICIES + policy;
}

// Persistent grid: as many workgroups as fit on the device at once (LDS and the
// 4-waves-per-SIMD register budget of k_jobs), never more than there are tiles.
static int persistent_grid(const JobsPlan &jp)
{
    int dev = 0, ncu = 256;
    size_t lds_cu = 160 * 1024;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) {
        ncu = prop.multiProcessorCount;
        if (prop.maxSharedMemoryPerMultiProcessor > 0) lds_cu = prop.maxSharedMemoryPerMultiProcessor;
    }
    const int by_waves = (4 * 4 * 64) / JOB_THREADS;   // 4 waves per SIMD, 4 SIMDs per CU
    const int by_lds = (int)(lds_cu / std::max<size_t>(jp.lds_max, 1));
    const int per_cu = std::max(1, std::min(by_waves, by_lds));
    return (int)std::max<long>(1, std::min<long>((long)ncu * per_cu, (long)jp.tiles->first[1]));
}

static hipError_t enqueue_jobs(const JobsPlan &jp, unsigned char *ws, int persistent, hipStream_t s)
{
    unsigned int *next = reinterpret_cast<unsigned int *>(ws);
    const JobDesc *jobs = reinterpret_cast<const JobDesc *>(ws + HEADER_BYTES);
    const TileDesc *tiles = reinterpret_cast<const TileDesc *>(ws + HEADER_BYTES +
                                                               jp.jobs.size() * sizeof(JobDesc));
    const int *first = jp.tiles->first;
    if (persistent) hipLaunchKernelGGL(k_reset_queue, dim3(1), dim3(64), 0, s, next);
    // the Gram form's kernels, the most users (and the longest tiles) first, then the residual's
    for (int k = N_JOB_KERNELS - 1; k >= 1; --k) {
        if (first[k] == first[k + 1]) continue;
        const hipError_t e = launch_jobs_gram(k, jp.f16, jp.box, jobs, tiles + first[k], next + k,
                                              first[k + 1] - first[k], persistent, s);
        if (e != hipSuccess) return e;
    }
    const int ntiles = first[1];
    if (ntiles == 0) return hipSuccess;
    const int grid = persistent ? persistent_grid(jp) : ntiles;
    if (jp.f16) {
        if (jp.box) hipLaunchKernelGGL((k_jobs<true, true>), dim3(grid), dim3(JOB_THREADS), jp.lds_max, s, jobs, tiles, next, ntiles, persistent);
        else hipLaunchKernelGGL((k_jobs<true, false>), dim3(grid), dim3(JOB_THREADS), jp.lds_max, s, jobs, tiles, next, ntiles, persistent);
    } else {
        if (jp.box) hipLaunchKernelGGL((k_jobs<false, true>), dim3(grid), dim3(JOB_THREADS), jp.lds_max, s, jobs, tiles, next, ntiles, persistent);
        else hipLaunchKernelGGL((k_jobs<false, false>), dim3(grid), dim3(JOB_THREADS), jp.lds_max, s, jobs, tiles, next, ntiles, persistent);
    }
    return hipGetLastError();
}

static const void *jobs_kernel(bool f16, bool box)
{
    if (f16) return box ? reinterpret_cast<const void *>(k_jobs<true, true>)
                        : reinterpret_cast<const void *>(k_jobs<true, false>);
    return box ? reinterpret_cast<const void *>(k_jobs<false, true>)
               : reinterpret_cast<const void *>(k_jobs<false, false>);
}

// Uploads the tables through the library's pinned buffer for this workspace,
// unless the workspace already holds exactly these bytes.
static hipError_t upload_tables(const JobsPlan &jp, unsigned char *ws, hipStream_t s)
{
    const size_t nj = jp.jobs.size() * sizeof(JobDesc), nt = jp.tiles->tiles.size() * sizeof(TileDesc);
    const size_t bytes = nj + nt;
    Staging &st = g_staging[ws];
    if (st.last_tiles == jp.tiles && st.last_jobs.size() == nj &&
        std::memcmp(st.last_jobs.data(), jp.jobs.data(), nj) == 0)
        return hipSuccess;
    hipError_t e = hipSuccess;
    if (st.uploaded) {
        e = hipEventSynchronize(st.uploaded);   // the last copy from this buffer is done
        if (e != hipSuccess) return e;
    } else {
        e = hipEventCreateWithFlags(&st.uploaded, hipEventDisableTiming);
        if (e != hipSuccess) return e;
    }
    if (st.bytes < bytes) {
        if (st.pinned) (void)hipHostFree(st.pinned);
        st.pinned = nullptr;
        st.bytes = 0;
        e = hipHostMalloc(&st.pinned, bytes, hipHostMallocDefault);
        if (e != hipSuccess) return e;
        st.bytes = bytes;
    }
    unsigned char *h = static_cast<unsigned char *>(st.pinned);
    std::memcpy(h, jp.jobs.data(), nj);
    std::memcpy(h + nj, jp.tiles->tiles.data(), nt);
    e = hipMemcpyAsync(ws + HEADER_BYTES, h, bytes, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    st.last_jobs.assign(h, h + nj);
    st.last_tiles = jp.tiles;
    return hipEventRecord(st.uploaded, s);
}

static void fill_pointers(JobsPlan &jp, const void *const *H, const void *const *y,
                          float *const *z, float *const *llr)
{
    for (size_t j = 0; j < jp.jobs.size(); ++j) {
        Params &P = jp.jobs[j].P;
        P.H = H[j];
        P.y = y[j];
        P.z = z ? reinterpret_cast<float2 *>(z[j]) : nullptr;
        P.llr = llr ? llr[j] : nullptr;
        P.z_hist = nullptr;
        P.lambda = nullptr;
        P.g_in = P.dinv_in = P.p_in = nullptr;
        ocd_problem pb;
        pb.B = P.B;
        pb.storage = jp.f16 ? OCD_STORE_F16 : OCD_STORE_F32;
        set_vec_ok(P, &pb, P.H, P.y);
    }
}

static std::string jobs_hash(const ocd_problem *jobs, int n)
{
    unsigned long long h = 1469598103934665603ULL;
    auto mix = [&](long long v) { h = (h ^ (unsigned long long)v) * 1099511628211ULL; };
    for (int j = 0; j < n; ++j) {
        const ocd_problem &p = jobs[j];
        mix(p.B); mix(p.U); mix(p.W); mix(p.S); mix(p.Q); mix(p.K); mix(p.mode); mix(p.storage);
    }
    char buf[64];
    std::snprintf(buf, sizeof buf, "%016llx|%d", h, n);
    return buf;
}

static ocd_status run_choice(const ocd_problem *jobs, int n, int choice, const void *const *H,
                             const void *const *y, float *const *z, float *const *llr,
                             unsigned char *ws, size_t ws_bytes, bool use_graph, hipStream_t s)
{
    JobsPlan jp;
    ocd_status st = plan_jobs(jobs, n, choice_policy(choice), choice_lane_mode(choice), jp);
    if (st != OCD_OK) return st;
    if (HEADER_BYTES + table_bytes(jp) > ws_bytes) return OCD_EINVAL;
    if (jp.tiles->tiles.empty()) return OCD_OK;
    fill_pointers(jp, H, y, z, llr);
    const void *fn = jobs_kernel(jp.f16, jp.box);
    if (jp.lds_max > 65536 &&
        hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)jp.lds_max) != hipSuccess)
        return OCD_EDEVICE;
    const int persistent = choice_persistent(choice);
    if (upload_tables(jp, ws, s) != hipSuccess) return OCD_EDEVICE;
    if (!use_graph) return enqueue_jobs(jp, ws, persistent, s) == hipSuccess ? OCD_OK : OCD_EDEVICE;

    char key[256];
    const int *first = jp.tiles->first;
    std::snprintf(key, sizeof key, "%p|%zu|%d|%d|%d|%d|%zu|%d|%d|%d", (void *)ws, jp.jobs.size(),
                  first[1], first[2], first[3], first[4], jp.lds_max, choice, (int)jp.f16,
                  (int)jp.box);
    auto it = g_graphs.find(key);
    if (it == g_graphs.end()) {
        if (!g_capture_stream &&
            hipStreamCreateWithFlags(&g_capture_stream, hipStreamNonBlocking) != hipSuccess)
            return OCD_EDEVICE;
        GraphEntry ge;
        if (hipStreamBeginCapture(g_capture_stream, hipStreamCaptureModeThreadLocal) != hipSuccess)
            return OCD_EDEVICE;
        hipError_t e = enqueue_jobs(jp, ws, persistent, g_capture_stream);
        hipError_t e2 = hipStreamEndCapture(g_capture_stream, &ge.graph);
        if (e != hipSuccess || e2 != hipSuccess) {
            if (ge.graph) (void)hipGraphDestroy(ge.graph);
            return OCD_EDEVICE;
        }
        if (hipGraphInstantiate(&ge.exec, ge.graph, nullptr, nullptr, 0) != hipSuccess) {
            (void)hipGraphDestroy(ge.graph);
            return OCD_EDEVICE;
        }
        it = g_graphs.emplace(key, ge).first;
    }
    return hipGraphLaunch(it->second.exec, s) == hipSuccess ? OCD_OK : OCD_EDEVICE;
}

}  // namespace ocd

using namespace ocd;

extern "C" size_t ocd_jobs_workspace_bytes(const ocd_problem *jobs, int n_jobs)
{
    size_t best = 0;
    for (int policy = 0; policy < N_POLICIES; ++policy)
        for (int mode = 0; mode < N_LANE_MODES; ++mode) {
            JobsPlan jp;
            if (plan_jobs(jobs, n_jobs, policy, mode, jp) != OCD_OK) return 0;
            best = std::max(best, HEADER_BYTES + table_bytes(jp));
        }
    return best;
}

extern "C" ocd_status ocd_detect_jobs(const ocd_problem *jobs, const void *const *H,
                                      const void *const *y, float *const *z, float *const *llr,
                                      int n_jobs, void *workspace, size_t workspace_bytes, int flags,
                                      hipStream_t stream)
{
    if (!jobs || n_jobs < 1 || !H || !y || !workspace) return OCD_EINVAL;
    if (reinterpret_cast<uintptr_t>(workspace) % 256) return OCD_EINVAL;
    for (int j = 0; j < n_jobs; ++j) {
        ocd_status st = validate(&jobs[j]);
        if (st != OCD_OK) return st;
        if (jobs[j].W > 0 && (!H[j] || !y[j])) return OCD_EINVAL;
    }
    std::lock_guard<std::mutex> lk(g_mu);
    unsigned char *ws = static_cast<unsigned char *>(workspace);
    const std::string hk = jobs_hash(jobs, n_jobs);
    int choice = DEFAULT_CHOICE;
    auto pit = g_choice.find(hk);
    if (pit != g_choice.end()) choice = pit->second;
    if (flags & OCD_JOBS_TUNE) {
        // batch tuner: time every (schedule, tile policy) on the caller's buffers
        hipEvent_t e0, e1;
        if (hipEventCreate(&e0) != hipSuccess) return OCD_EDEVICE;
        if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return OCD_EDEVICE; }
        // three launches of a choice, timed (ms; < 0 if the choice does not run)
        auto time_choice = [&](int c) -> float {
            ocd_status st = OCD_OK;
            (void)hipEventRecord(e0, stream);
            for (int rep = 0; rep < 3 && st == OCD_OK; ++rep)
                st = run_choice(jobs, n_jobs, c, H, y, z, llr, ws, workspace_bytes, false, stream);
            (void)hipEventRecord(e1, stream);
            if (st != OCD_OK || hipEventSynchronize(e1) != hipSuccess) return -1.f;
            float ms = 0.f;
            (void)hipEventElapsedTime(&ms, e0, e1);
            return ms;
        };
        // tile policies and lane modes shape the residual form's tiles only
        bool residual = false;
        for (int j = 0; j < n_jobs; ++j)
            residual |= !gram_form(jobs[j].B, jobs[j].U, jobs[j].W, jobs[j].S, jobs[j].K);
        std::vector<std::pair<float, int>> ranked;
        for (int c = 0; c < N_CHOICES; ++c) {
            if (!residual && (choice_lane_mode(c) != 0 ||
                              choice_policy(c) != choice_policy(DEFAULT_CHOICE)))
                continue;
            if (run_choice(jobs, n_jobs, c, H, y, z, llr, ws, workspace_bytes, false, stream) != OCD_OK)
                continue;
            const float ms = time_choice(c);
            if (ms >= 0.f) ranked.push_back({ms, c});
        }
        // the fastest three again, in three interleaved rounds: the lowest median
        // wins (the schedules are often within a few percent of each other)
        int best = choice;
        if (!ranked.empty()) {
            std::sort(ranked.begin(), ranked.end());
            const int nf = (int)std::min<size_t>(3, ranked.size());
            float t[3][3] = {};
            for (int rd = 0; rd < 3; ++rd)
                for (int k = 0; k < nf; ++k) {
                    const int f = rd % 2 ? nf - 1 - k : k;
                    t[f][rd] = time_choice(ranked[f].second);
                }
            float best_med = 1e30f;
            for (int f = 0; f < nf; ++f) {
                std::sort(t[f], t[f] + 3);
                if (t[f][0] >= 0.f && t[f][1] < best_med) { best_med = t[f][1]; best = ranked[f].second; }
            }
        }
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        choice = best;
        g_choice[hk] = choice;
    }
    if (flags & OCD_JOBS_PERSISTENT)
        choice = make_choice(choice_lane_mode(choice), 1, choice_policy(choice));
    const int forced_mode = (flags >> OCD_JOBS_LANE_MODE_SHIFT) & 3;
    if (forced_mode > N_LANE_MODES) return OCD_EINVAL;
    if (forced_mode)
        choice = make_choice(forced_mode - 1, choice_persistent(choice), choice_policy(choice));
    return run_choice(jobs, n_jobs, choice, H, y, z, llr, ws, workspace_bytes,
                      (flags & OCD_JOBS_GRAPH) != 0, stream);
}

extern "C" ocd_status ocd_jobs_schedule(const ocd_problem *jobs, int n_jobs, int *persistent,
                                        int *tile_policy, int *lane_mode)
{
    if (!jobs || n_jobs < 1 || !persistent || !tile_policy || !lane_mode) return OCD_EINVAL;
    for (int j = 0; j < n_jobs; ++j) {
        ocd_status st = validate(&jobs[j]);
        if (st != OCD_OK) return st;
    }
    std::lock_guard<std::mutex> lk(g_mu);
    int choice = DEFAULT_CHOICE;
    auto it = g_choice.find(jobs_hash(jobs, n_jobs));
    if (it != g_choice.end()) choice = it->second;
    *persistent = choice_persistent(choice);
    *tile_policy = choice_policy(choice);
    *lane_mode = choice_lane_mode(choice);
    return OCD_OK;
}

extern "C" void ocd_release_graphs(void)
{
    std::lock_guard<std::mutex> lk(g_mu);
    for (auto &kv : g_graphs) {
        if (kv.second.exec) (void)hipGraphExecDestroy(kv.second.exec);
        if (kv.second.graph) (void)hipGraphDestroy(kv.second.graph);
    }
    g_graphs.clear();
    for (auto &kv : g_staging) {
        if (kv.second.uploaded) {
            (void)hipEventSynchronize(kv.second.uploaded);
            (void)hipEventDestroy(kv.second.uploaded);
        }
        if (kv.second.pinned) (void)hipHostFree(kv.second.pinned);
    }
    g_staging.clear();
    std::lock_guard<std::mutex> lt(g_tiles_mu);
    g_tiles.clear();
}
