// ocd_gram.hip -- the detection kernel for channels that several symbols share
// (ocd_gram.h): one workgroup per subcarrier and per 16 symbols of it.
#include "ocd_gram.h"

namespace ocd {

// VEC: rows of even length, aligned.  HALF: see gram_dispatch.  NW: see gram_waves.
template <int UP, GramSymbols SY, bool F16, bool BOX, bool VEC, bool HALF, int NW>
__global__ __launch_bounds__(GRAM_THREADS, UP == 32 ? 3 : 2) void k_gram(Params P, int tiles)
{
    using M = GramLds<UP, SY, NW>;
    __shared__ __align__(16) double lds[M::DOUBLES];
    __shared__ GramUser us[M::SG * UP];
    stagger_loads(P);
    const int g = tiles == 1 ? (int)blockIdx.x : (int)blockIdx.x / tiles;
    const int s0 = tiles == 1 ? 0 : 16 * ((int)blockIdx.x - g * tiles);
    const int ns = min(16, P.S - s0);
    gram_tile<UP, SY, F16, BOX, VEC, HALF, NW>(P, (long)g * M::SG, s0, ns, lds, us);
}

template <int UP, GramSymbols SY, bool F16, bool BOX, bool VEC, bool HALF, int NW>
static hipError_t launch_gram_k(const Params &p, hipStream_t s)
{
    auto fn = k_gram<UP, SY, F16, BOX, VEC, HALF, NW>;
    constexpr int SG = GramLds<UP, SY, NW>::SG;
    const int tiles = (p.S + 15) / 16;
    // nearly always one launch; else whole groups of SG subcarriers each
    const long most = groups_per_launch(tiles, GRAM_THREADS) * SG;
    if (p.W > most) {
        constexpr size_t c = F16 ? 4 : 8;   // bytes of an entry of H and y
        for (long w0 = 0; w0 < p.W; w0 += most) {
            Params q = p;
            const long v0 = w0 * p.S, d0 = w0 * (p.per_sweep ? p.K : 1) * p.U;
            q.W = (int)(p.W - w0 < most ? p.W - w0 : most);
            q.H = static_cast<const unsigned char *>(p.H) + (size_t)w0 * p.U * p.B * c;
            q.y = static_cast<const unsigned char *>(p.y) + (size_t)v0 * p.B * c;
            if (p.g_in) q.g_in = p.g_in + w0 * p.U;
            if (p.dinv_in) q.dinv_in = p.dinv_in + d0;
            if (p.p_in) q.p_in = p.p_in + d0;
            if (p.z) q.z = p.z + v0 * p.U;
            if (p.llr) q.llr = p.llr + v0 * p.U * p.Q;
            if (p.z_hist) q.z_hist = p.z_hist + v0 * p.K * p.U;
            const hipError_t e = launch_gram_k<UP, SY, F16, BOX, VEC, HALF, NW>(q, s);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    Params q = p;
    if (q.stagger > 0) {
        int per_cu = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per_cu, reinterpret_cast<const void *>(fn), GRAM_THREADS, 0);
        if (e != hipSuccess) return e;
        q.stagger_cap = per_cu * device_cu_count();
    }
    hipLaunchKernelGGL(fn, dim3((unsigned)((p.W + SG - 1) / SG) * tiles), dim3(GRAM_THREADS), 0, s,
                       q, tiles);
    return hipGetLastError();
}

template <int UP, GramSymbols SY, bool F16, bool BOX, bool VEC, bool HALF>
static hipError_t launch_gram_w(const Params &p, hipStream_t s)
{
    if constexpr (UP <= 16) {
        if (gram_waves(p.B, p.U, p.S, (long)p.W * ((p.S + 15) / 16)) == 1)
            return launch_gram_k<UP, SY, F16, BOX, VEC, HALF, 1>(p, s);
    }
    return launch_gram_k<UP, SY, F16, BOX, VEC, HALF, 4>(p, s);
}

template <int UP, GramSymbols SY, bool F16, bool BOX>
static hipError_t launch_gram_c(const Params &p, hipStream_t s)
{
    return gram_dispatch<UP, F16>(p, [&](auto vec, auto half) {
        return launch_gram_w<UP, SY, F16, BOX, vec(), half()>(p, s);
    });
}

template <int UP, GramSymbols SY>
static hipError_t launch_gram_s(bool f16, const Params &p, hipStream_t s)
{
    if (f16) return p.box ? launch_gram_c<UP, SY, true, true>(p, s)
                          : launch_gram_c<UP, SY, true, false>(p, s);
    return p.box ? launch_gram_c<UP, SY, false, true>(p, s)
                 : launch_gram_c<UP, SY, false, false>(p, s);
}

template <int UP>
static hipError_t launch_gram_u(bool f16, const Params &p, hipStream_t s)
{
    return p.S <= 8 ? launch_gram_s<UP, SY_8>(f16, p, s) : launch_gram_s<UP, SY_16>(f16, p, s);
}

hipError_t launch_gram(bool f16, const Params &p, hipStream_t s)
{
    if (p.U <= 8) return launch_gram_u<8>(f16, p, s);
    if (p.U <= 16) return launch_gram_u<16>(f16, p, s);
    return launch_gram_u<32>(f16, p, s);
}

}  // namespace ocd
