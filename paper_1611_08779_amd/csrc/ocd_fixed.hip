// ocd_fixed.hip -- Algorithm 1 in the fixed-point datapath of Section IV-C, for
// comparing the paper's 16-bit design with floating point on the same inputs.
//
// Words (H, y, the residual r, z, beta, d^-1, p) are 16-bit two's complement with
// 11 fractional bits (Q5.11).  Products of two words are exact; the inner
// products are exact 64-bit sums of them (the paper's 36-bit adder tree, which
// they fit on any input whose sums stay in 36 bits).  ||h_u||^2 + alpha and
// h_u^H r are shifted right by b = ceil(log2 B); the two shifts cancel in
// d^-1 h^H r.  The reciprocal d^-1 comes from normalising its input to [1/2, 1),
// indexing a 2048-entry table of 18-bit normalised reciprocals with the 11 bits
// after the leading one, and shifting back.  Every narrowing to 16 bits rounds
// half up and saturates.  The paper's design has no soft-output unit: the LLRs
// are formed in FP32 from the fixed-point z and p, as in the floating-point path.
//
// Two forms: tiles of 16 symbols on the integer matrix cores (k_fixed_tile) and, for few
// symbols a subcarrier or many antennas, lane groups (k_forward_fx).
//
// Lane groups: L lanes per vector; lane j holds residual entries b = j + L i.  The
// updates run in FP64 on integer values: every intermediate of the datapath is an integer below 2^53 (products below 2^32, sums below 2^41,
// d^-1 times a shifted inner product below 2^51), so every FP64 operation on them
// is exact, a floor after a power-of-two scale is the arithmetic shift, and
// clamps are the saturation; MI355X runs FP64 FMAs at the FP32 vector rate.  The
// sums are exact, so the order of the cross-lane sums does not matter and the
// result is bit-exact.  The H_w a workgroup touches are staged in LDS once, their
// int16 values held exactly in FP32 (where they fit in 32 KB), so that an update's
// column read is an LDS read rather than a round trip to the L2, and each entry
// reaches FP64 in one conversion.
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "ocd_api_internal.h"
#include "ocd_stage.h"

namespace ocd {

struct FxParams {
    int B, U, W, S, K, Q, box, b;
    long long lam_q;    // alpha in Q.22
    int beta_fx;        // box half-width in Q.11
    float lam, Es, N0, sqEs, qscale;
    const int16_t *H;   // [W][U][B][2]
    const int16_t *y;   // [W][S][B][2]
    int16_t *z;         // [W][S][U][2] or nullptr
    float *llr;         // [W][S][U][Q] or nullptr
};

__device__ __forceinline__ long long fx_sat16(long long v)
{
    return v < -32768 ? -32768 : (v > 32767 ? 32767 : v);
}

// v / 2^s rounded half up (s >= 1)
__device__ __forceinline__ long long fx_round_shift(long long v, int s)
{
    return (v + (1ll << (s - 1))) >> s;
}

// Q.11 reciprocal of x > 0 given in Q.22 units: normalise, index the table with
// the 11 bits after the leading one, denormalise; 0 for x <= 0.  The table entry
// round(2^18 / (1 + (i + 1/2) / 2048)) is evaluated where it is needed (IEEE
// double division is correctly rounded, so it is the table's value).
__device__ __forceinline__ long long fx_recip(long long x)
{
    if (x <= 0) return 0;
    const int n = 64 - __clzll(x);   // bit length
    const long long idx = n >= 12 ? (x >> (n - 12)) & 2047 : (x << (12 - n)) & 2047;
    const long long lut = (long long)floor(262144.0 / (1.0 + ((double)idx + 0.5) / 2048.0) + 0.5);
    const long long d = (16 - n >= 0) ? lut * (1ll << (16 - n)) : fx_round_shift(lut, n - 16);
    return fx_sat16(d);
}

// A 64-bit lane value from another lane of the row: the DPP move of both halves.
template <int CTRL>
__device__ __forceinline__ long long dpp_get_i64(long long x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)x, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), CTRL, 0xF, 0xF, false);
    return (long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// Exact FP64 helpers on integer values (see the header).
__device__ __forceinline__ double fx_sat16d(double v) { return fmin(fmax(v, -32768.0), 32767.0); }

// v / 2^s rounded half up: floor((v + 2^(s-1)) 2^-s), exact for integer v < 2^53
__device__ __forceinline__ double fx_round_shiftd(double v, double half, double inv)
{
    return floor((v + half) * inv);
}

template <int CTRL>
__device__ __forceinline__ double dpp_get_f64(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// Sum over the L lanes of an aligned group (L = 16 or 32), the same in every lane;
// the values are integers below 2^53, so every partial sum is exact.
template <int L>
__device__ __forceinline__ double group_sum_f64(double x)
{
    x += dpp_get_f64<DPP_QUAD_XOR1>(x);
    x += dpp_get_f64<DPP_QUAD_XOR2>(x);
    x += dpp_get_f64<DPP_ROW_HALF_MIRROR>(x);
    x += dpp_get_f64<DPP_ROW_MIRROR>(x);
    if constexpr (L >= 32) x += __shfl_xor(x, 16, 32);
    return x;
}

// Exact sum over the L lanes of an aligned group (L = 16 or 32), the same in
// every lane; integer addition is associative, so the order does not matter.
template <int L>
__device__ __forceinline__ long long group_sum_i64(long long x)
{
    x += dpp_get_i64<DPP_QUAD_XOR1>(x);
    x += dpp_get_i64<DPP_QUAD_XOR2>(x);
    x += dpp_get_i64<DPP_ROW_HALF_MIRROR>(x);
    x += dpp_get_i64<DPP_ROW_MIRROR>(x);
    if constexpr (L >= 32) x += __shfl_xor(x, 16, 32);
    return x;
}

// The LLRs of component ax (value zv, Q.11) of a user, whose entry o of [W][S][U] is given.
__device__ __forceinline__ void fx_axis_llrs(const FxParams &P, float p, long long gi, int zv, int ax,
                                             size_t o)
{
    const int half = P.Q >> 1;
    const float g = (float)gi * (1.0f / 4194304.0f);
    float mu, rho;
    if (P.lam > 0.f) {
        mu = p * (1.0f / 2048.0f);
        rho = g / P.lam;
    } else {
        mu = 1.0f;
        rho = g * P.Es / P.N0;
    }
    float a = 0.f, c = 0.f;
    if (mu > 0.f && rho > 0.f) {
        a = 1.0f / (mu * P.sqEs * P.qscale);
        c = rho * P.qscale * P.qscale;
    }
    const float t = (float)zv * (1.0f / 2048.0f) * a;
    float *dst = P.llr + o * P.Q + ax * half;
    if (half == 3) axis_llrs<3>(t, c, dst);
    else if (half == 2) axis_llrs<2>(t, c, dst);
    else axis_llrs<1>(t, c, dst);
}

// STAGED: the H_w of the subcarriers a workgroup touches are copied into LDS once
// (int16 values held exactly in FP32), and every update reads its column there;
// otherwise (channels too large for the LDS budget) each update reads its column
// from global memory, where the S symbols of a subcarrier share it through the
// caches.  The arithmetic is the same either way.
template <int L, int NPL, bool STAGED>
__global__ __launch_bounds__(256) void k_forward_fx(FxParams P)
{
    constexpr int G = 256 / L;
    __shared__ int zs[G][32][2];
    __shared__ int ds[G][32], ps[G][32];
    __shared__ long long gs[G][32];
    extern __shared__ __align__(16) float2 hst[];    // STAGED: [slots][U][B] int16 values in FP32
    const int grp = threadIdx.x / L, j = threadIdx.x % L;
    const long v = (long)blockIdx.x * G + grp;
    const long nvec = (long)P.W * P.S;
    const int U = P.U, B = P.B, b = P.b;
    const float2 *Hs = nullptr;
    if constexpr (STAGED) {
        const long v0 = (long)blockIdx.x * G, vl = (v0 + G < nvec ? v0 + G : nvec) - 1;
        const long w_first = v0 / P.S;
        const int total = (int)(vl / P.S - w_first + 1) * U * B;
        const uint32_t *src = reinterpret_cast<const uint32_t *>(P.H) + (size_t)w_first * U * B;
        for (int i = threadIdx.x; i < total; i += blockDim.x) {
            const uint32_t e = src[i];
            hst[i] = make_float2((float)(int16_t)(e & 0xFFFFu), (float)(int16_t)(e >> 16));
        }
        __syncthreads();
        Hs = hst + (size_t)((v < nvec ? v : v0) / P.S - w_first) * U * B;
    }
    if (v >= nvec) return;   // a whole lane group at once
    const int16_t *Hw = P.H + (size_t)(v / P.S) * U * B * 2;
    const int16_t *yv = P.y + (size_t)v * B * 2;

    double rr[NPL], ri[NPL];   // residual entries j + L i, Q.11 integers
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
        const int a = j + L * i;
        rr[i] = a < B ? (double)yv[2 * a] : 0.0;
        ri[i] = a < B ? (double)yv[2 * a + 1] : 0.0;
    }

    // preprocessing (Alg. 1, initialisation): ||h_u||^2, d_u^-1, p_u
    for (int u = 0; u < U; ++u) {
        const int16_t *hu = Hw + (size_t)u * B * 2;
        long long g = 0;
#pragma unroll
        for (int i = 0; i < NPL; ++i) {
            const int a = j + L * i;
            if (a < B) {
                const long long hr = hu[2 * a], hi = hu[2 * a + 1];
                g += hr * hr + hi * hi;
            }
        }
        g = group_sum_i64<L>(g);
        if (j == 0) {
            const long long d = fx_recip((g + P.lam_q) >> b);
            gs[grp][u] = g;
            ds[grp][u] = (int)d;
            ps[grp][u] = (int)fx_sat16(fx_round_shift(d * (g >> b), 22));
            zs[grp][u][0] = 0;
            zs[grp][u][1] = 0;
        }
    }
    __builtin_amdgcn_wave_barrier();

    // column entries as (re, im) int16 pairs in one dword; lanes past B hold 0
    auto load_col = [&](int u, uint32_t (&h)[NPL]) {
        const uint32_t *hu = reinterpret_cast<const uint32_t *>(Hw) + (size_t)u * B;
#pragma unroll
        for (int i = 0; i < NPL; ++i) {
            const int a = j + L * i;
            h[i] = a < B ? hu[a] : 0u;
        }
    };
    // the same column from the staged copy (int16 values held exactly in FP32)
    auto load_col_s = [&](int u, float2 (&h)[NPL]) {
        const float2 *hu = Hs + (size_t)u * B;
#pragma unroll
        for (int i = 0; i < NPL; ++i) {
            const int a = j + L * i;
            h[i] = a < B ? hu[a] : make_float2(0.f, 0.f);
        }
    };
    const double inv_b = ldexp(1.0, -b);
    uint32_t hn[NPL];
    float2 hf[NPL];
    if constexpr (STAGED) load_col_s(0, hf);
    else load_col(0, hn);
    for (int k = 0; k < P.K; ++k)
        for (int u = 0; u < U; ++u) {
            double hr[NPL], hi[NPL];
#pragma unroll
            for (int i = 0; i < NPL; ++i) {
                hr[i] = STAGED ? (double)hf[i].x : (double)(int16_t)(hn[i] & 0xFFFFu);
                hi[i] = STAGED ? (double)hf[i].y : (double)(int16_t)(hn[i] >> 16);
            }
            // the next update's column is in flight while this one computes
            if constexpr (STAGED) load_col_s(u + 1 < U ? u + 1 : 0, hf);
            else load_col(u + 1 < U ? u + 1 : 0, hn);
            double ire = 0.0, iim = 0.0;   // h_u^H r, Q.22 integers
#pragma unroll
            for (int i = 0; i < NPL; ++i) {
                ire = fma(hr[i], rr[i], fma(hi[i], ri[i], ire));
                iim = fma(hr[i], ri[i], fma(-hi[i], rr[i], iim));
            }
            ire = floor(group_sum_f64<L>(ire) * inv_b);   // arithmetic shift by b
            iim = floor(group_sum_f64<L>(iim) * inv_b);
            const double d = ds[grp][u], p = ps[grp][u];
            const double zr = zs[grp][u][0], zi = zs[grp][u][1];
            // c = d^-1 h^H r + p z in Q.33, narrowed to Q.11
            const double h22 = 2097152.0, i22 = 1.0 / 4194304.0;
            double cre = fx_sat16d(fx_round_shiftd(fma(d, ire, p * zr * 2048.0), h22, i22));
            double cim = fx_sat16d(fx_round_shiftd(fma(d, iim, p * zi * 2048.0), h22, i22));
            if (P.box) {
                const double bt = P.beta_fx;
                cre = fmin(fmax(cre, -bt), bt);
                cim = fmin(fmax(cim, -bt), bt);
            }
            // r - round(h (c - z) / 2^11), each component saturated.  The 2^-11 is
            // folded into (c - z): every product and partial sum is then an integer
            // times 2^-11 below 2^22, exact in FP64, so the floor sees the same value
            // as with the scale applied after the sum.
            const double dre = (cre - zr) * (1.0 / 2048.0), dim = (cim - zi) * (1.0 / 2048.0);
#pragma unroll
            for (int i = 0; i < NPL; ++i) {
                const double tr = floor(fma(hr[i], dre, fma(-hi[i], dim, 0.5)));
                const double ti = floor(fma(hr[i], dim, fma(hi[i], dre, 0.5)));
                rr[i] = fx_sat16d(rr[i] - tr);
                ri[i] = fx_sat16d(ri[i] - ti);
            }
            __builtin_amdgcn_wave_barrier();   // every lane has read z_u
            if (j == 0) {
                zs[grp][u][0] = (int)cre;
                zs[grp][u][1] = (int)cim;
            }
            __builtin_amdgcn_wave_barrier();
        }

    // outputs: lane pair index idx = 2u + axis
    for (int idx = j; idx < 2 * U; idx += L) {
        const int u = idx >> 1, ax = idx & 1;
        const int zv = zs[grp][u][ax];
        if (P.z) P.z[(size_t)v * U * 2 + idx] = (int16_t)zv;
        if (P.llr) fx_axis_llrs(P, (float)ps[grp][u], gs[grp][u], zv, ax, (size_t)v * U + u);
    }
}

// Many symbols of one subcarrier at once: the sums h_u^H r on the matrix cores.  A tile
// is a subcarrier and up to 16 of its symbols, taken by NW waves with NBW blocks of 32
// antennas each; lane l holds residual entries 8 (l / 16) .. + 7 of each block for symbol
// l mod 16, int16 pairs.  Words are split into bytes, r = 256 rh + rl (rl unsigned, given
// to the signed unit as rl - 128, and 128 sum(h) added back through the accumulator's
// start) and h = 256 hh + hl (both signed), so that h_u^H r is four int32 sums of byte
// products (v_mfma_i32_16x16x64_i8: rows Re hh, Re hl, Im hh, Im hl; columns symbols),
// which are exact and already summed over the lanes.  An hh of 128 (h >= 32640, or its
// negative in the Im row) does not fit a byte: a workgroup that stages one takes the sums
// in FP64 instead.  The update r - round(h (c - z) / 2^11) is (2^11 r + 1023 - h (c - z))
// >> 11, two v_dot2_i32_i16 a component; where some |c - z| >= 2^14 its sum could leave 32
// bits, and the rest of the tile's updates are done in FP64.
//
// Bound by the vector issue (90% busy at 4000 subcarriers): per antenna four products, two
// shifts, a narrowing and the byte split, 33 cycles a wave, and some 50 instructions an
// update for the rest; with few tiles by the latency of an update (0.6 us).  NW and NBW: 16
// entries a lane balance the two (B = 128, 1200 x 14 vectors: one wave 47 us, two 42, four
// 45; B = 256, U = 16: 310, 224, 144).  1200 x 14 vectors of 128 x 8, K = 3: 70.5 us in lane
// groups with FP64 sums, 35.6 so.
struct FxUser {
    double d, p;
    long long g;
    int2 start[2];    // 128 sum(h) of the rows hh, hl of Re and Im
};

// LDS: per user and 8 antennas the four rows' bytes (64) and the int16 pairs (32); the
// users' constants; every lane's z; partial sums of the waves (two updates in turn).
template <int NBW, int NW>
struct FxTile {
    static constexpr int CHUNKS = 4 * NBW * NW, THREADS = 64 * NW;
    __host__ __device__ static size_t users(int U) { return (size_t)U * CHUNKS * 96; }
    __host__ __device__ static size_t z(int U) { return users(U) + U * sizeof(FxUser); }
    __host__ __device__ static size_t sums(int U) { return z(U) + (size_t)U * THREADS * 4; }
    __host__ __device__ static size_t bytes(int U)
    {
        return sums(U) + (NW > 1 ? 2 * NW * 32 * sizeof(double) : 0);
    }
};

__device__ __forceinline__ int fx_lo(uint32_t e) { return (int16_t)(e & 0xFFFFu); }
__device__ __forceinline__ int fx_hi(uint32_t e) { return (int16_t)(e >> 16); }
__device__ __forceinline__ uint32_t fx_pack(int re, int im)
{
    return ((uint32_t)re & 0xFFFFu) | ((uint32_t)im << 16);
}

// Eight consecutive entries from a of a row of B, zero past its end.
__device__ __forceinline__ void fx_load8(const uint32_t *row, int a, int B, bool vec,
                                         uint32_t (&e)[8])
{
    if (vec) {   // B a multiple of 4, rows 16-byte aligned
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            uint4 x = make_uint4(0, 0, 0, 0);
            if (a + 4 * q < B) x = *reinterpret_cast<const uint4 *>(row + a + 4 * q);
            e[4 * q] = x.x;
            e[4 * q + 1] = x.y;
            e[4 * q + 2] = x.z;
            e[4 * q + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) e[q] = a + q < B ? row[a + q] : 0u;
    }
}

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef short i16x2 __attribute__((ext_vector_type(2)));

// a . b + c, in the form that saturates (no sum here does): its c need not be the register
// of the result, so that a constant takes no copy, and it follows itself without a wait.
__device__ __forceinline__ int fx_dot2(uint32_t a, uint32_t b, int c)
{
    return __builtin_amdgcn_sdot2(__builtin_bit_cast(i16x2, a), __builtin_bit_cast(i16x2, b), c,
                                  true);
}

// The same value, not known to be: keeps what the rare branches derive from it out of the
// registers of the others.
__device__ __forceinline__ uint32_t fx_opaque(uint32_t x)
{
    asm("" : "+v"(x));
    return x;
}

template <int NBW, int NW>
__global__ __launch_bounds__(64 * NW, 4) void k_fixed_tile(FxParams P, int tiles, bool vec)
{
    using M = FxTile<NBW, NW>;
    extern __shared__ __align__(16) unsigned char fx_lds[];
    const int U = P.U, B = P.B, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int w = blockIdx.x / tiles, s0 = 16 * (blockIdx.x - w * tiles);
    const int ns = min(16, P.S - s0);
    const int sym = lane & 15, g = lane >> 4, comp = g & 1;   // comp: 0 for Re, 1 for Im
    const long v = (long)w * P.S + s0 + min(sym, ns - 1);
    FxUser *us = reinterpret_cast<FxUser *>(fx_lds + M::users(U));
    int *zs = reinterpret_cast<int *>(fx_lds + M::z(U)) + tid;
    double *sums = reinterpret_cast<double *>(fx_lds + M::sums(U));

    const uint32_t *yv = reinterpret_cast<const uint32_t *>(P.y) + (size_t)v * B;
    uint32_t r[8 * NBW];
#pragma unroll
    for (int m = 0; m < NBW; ++m) {
        uint32_t e[8];
        fx_load8(yv, 32 * (wave * NBW + m) + 8 * g, B, vec, e);
#pragma unroll
        for (int q = 0; q < 8; ++q) r[8 * m + q] = e[q];
    }

    // the channel's bytes and words, ||h_u||^2, d_u^-1, p_u: a lane takes 8 antennas of a
    // user at a time, CHUNKS neighbouring lanes a user
    bool wide = false;
    const uint32_t *Hw = reinterpret_cast<const uint32_t *>(P.H) + (size_t)w * U * B;
    const int items = (U * M::CHUNKS + M::THREADS - 1) / M::THREADS * M::THREADS;
    for (int it = tid; it < items; it += M::THREADS) {
        const int u = it / M::CHUNKS, c = it % M::CHUNKS;
        double gg = 0.0;
        int st[4] = {0, 0, 0, 0};
        if (u < U) {
            uint32_t e[8], rows[4][4];
            fx_load8(Hw + (size_t)u * B, 8 * c, B, vec, e);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int hr = fx_lo(e[q]), hi = fx_hi(e[q]);
                const int a[2] = {hr, -hi}, b[2] = {hi, hr};   // (first, second) of Re and Im
                gg = fma((double)hr, (double)hr, fma((double)hi, (double)hi, gg));
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    const int ah = (a[x] + 128) >> 8, bh = (b[x] + 128) >> 8;
                    const int al = a[x] - 256 * ah, bl = b[x] - 256 * bh;
                    wide |= (ah > 127) | (bh > 127);
                    st[2 * x] += ah + bh;
                    st[2 * x + 1] += al + bl;
                    const uint32_t ph = (ah & 255) | (bh & 255) << 8;
                    const uint32_t pl = (al & 255) | (bl & 255) << 8;
                    if (q & 1) {
                        rows[2 * x][q / 2] |= ph << 16;
                        rows[2 * x + 1][q / 2] |= pl << 16;
                    } else {
                        rows[2 * x][q / 2] = ph;
                        rows[2 * x + 1][q / 2] = pl;
                    }
                }
            }
            uint4 *o = reinterpret_cast<uint4 *>(fx_lds + (size_t)it * 64);
#pragma unroll
            for (int x = 0; x < 4; ++x)
                o[x] = make_uint4(rows[x][0], rows[x][1], rows[x][2], rows[x][3]);
            uint4 *o2 = reinterpret_cast<uint4 *>(fx_lds + (size_t)U * M::CHUNKS * 64 +
                                                  (size_t)it * 32);
            o2[0] = make_uint4(e[0], e[1], e[2], e[3]);
            o2[1] = make_uint4(e[4], e[5], e[6], e[7]);
        }
#pragma unroll
        for (int o = 1; o < M::CHUNKS; o *= 2) {
            gg += __shfl_xor(gg, o, 64);
#pragma unroll
            for (int x = 0; x < 4; ++x) st[x] += __shfl_xor(st[x], o, 64);
        }
        if (u < U && c == 0) {
            const long long gi = (long long)gg, d = fx_recip((gi + P.lam_q) >> P.b);
            us[u].d = (double)d;
            us[u].p = (double)fx_sat16(fx_round_shift(d * (gi >> P.b), 22));
            us[u].g = gi;
            us[u].start[0] = make_int2(128 * st[0], 128 * st[1]);
            us[u].start[1] = make_int2(128 * st[2], 128 * st[3]);
        }
    }
    for (int u = 0; u < U; ++u) zs[u * M::THREADS] = 0;   // each lane's own
    wide = __syncthreads_or(wide);

    const double inv_b = ldexp(1.0, -P.b);
    // rows 4 g, 4 g + 1 of the product, which lane group g gets: hh, hl of its component
    const unsigned char *abase =
        fx_lds + (4 * NBW * wave + g) * 64 + (((lane >> 2) & 1) * 2 + (lane & 1)) * 16;
    const int beta = P.box ? P.beta_fx : 32768;
    const int cmin = max(-32768, -beta), cmax = min(32767, beta);
    const unsigned char *wbase = fx_lds + (size_t)U * M::CHUNKS * 64 + (4 * NBW * wave + g) * 32;
    int end = P.K * U, n = 0, u = 0;
    auto load_h = [&](uint32_t (&h)[8 * NBW]) {
#pragma unroll
        for (int m = 0; m < NBW; ++m) {
            const uint4 *src =
                reinterpret_cast<const uint4 *>(wbase + (size_t)(u * M::CHUNKS + 4 * m) * 32);
            const uint4 x = src[0], y = src[1];
            h[8 * m] = x.x; h[8 * m + 1] = x.y; h[8 * m + 2] = x.z; h[8 * m + 3] = x.w;
            h[8 * m + 4] = y.x; h[8 * m + 5] = y.y; h[8 * m + 6] = y.z; h[8 * m + 7] = y.w;
        }
    };
    // the change of z_u (the lane's component) for the wave's part t of h_u^H r
    auto change = [&](double t, int z) {
        if constexpr (NW > 1) {
            double *sh = sums + (n & 1) * NW * 32;
            if (g < 2) sh[wave * 32 + lane] = t;
            __syncthreads();
#pragma unroll
            for (int x = 1; x < NW; ++x) t += sh[(wave ^ x) * 32 + (lane & 31)];
        }
        // c = d^-1 h^H r + p z in Q.33, narrowed to Q.11: the sum is shifted by b, and
        // c is below 2^29 before its narrowing
        t = fx_round_shiftd(fma(us[u].d, floor(t * inv_b), us[u].p * 2048.0 * z), 2097152.0,
                            1.0 / 4194304.0);
        return min(max((int)t, cmin), cmax) - z;
    };
    auto next = [&] { u = u + 1 < U ? u + 1 : 0; };

    if (!wide)
        for (; n < end; ++n, next()) {
            uint32_t h[8 * NBW];
            load_h(h);
            const int z = zs[u * M::THREADS];
            i32x4 ah = {0, 0, 0, 0}, al = {0, 0, 0, 0};
            if (wave == 0) {
                const int2 st = us[u].start[comp];
                al[0] = st.x;
                al[1] = st.y;
            }
#pragma unroll
            for (int m = 0; m < NBW; ++m) {
                const i32x4 a = *reinterpret_cast<const i32x4 *>(
                    abase + (size_t)(u * M::CHUNKS + 4 * m) * 64);
                i32x4 bh, bl;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t x = r[8 * m + 2 * q], y = r[8 * m + 2 * q + 1];
                    bh[q] = (int)__builtin_amdgcn_perm(y, x, 0x07050301u);
                    bl[q] = (int)(__builtin_amdgcn_perm(y, x, 0x06040200u) ^ 0x80808080u);
                }
                ah = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, bh, ah, 0, 0, 0);
                al = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, bl, al, 0, 0, 0);
            }
            const int dc = change(
                fma(65536.0, (double)ah[0], fma(256.0, (double)(ah[1] + al[0]), (double)al[1])), z);
            // the same in every wave of the workgroup
            if (!__all(max(dc, -dc) < 16384)) {
                ++n, ++end;   // again below, in the other place for the partial sums
                break;
            }
            zs[u * M::THREADS] = z + dc;
            const auto both = __builtin_amdgcn_permlane16_swap((unsigned)dc, (unsigned)dc, false, false);
            const int dr = (int)both[0], di = (int)both[1];
            const uint32_t nre = fx_pack(-dr, di), nim = fx_pack(-di, -dr);
            // products first, in the order given: a shift that follows its product waits
#pragma unroll
            for (int i = 0; i < 8 * NBW; i += 8) {
                int y[16];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    y[2 * q] = fx_dot2(h[i + q], nre, fx_dot2(r[i + q], 2048u, 1023));
                    y[2 * q + 1] = fx_dot2(h[i + q], nim, fx_dot2(r[i + q], 2048u << 16, 1023));
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    r[i + q] = __builtin_bit_cast(
                        uint32_t, __builtin_amdgcn_cvt_pk_i16(y[2 * q] >> 11, y[2 * q + 1] >> 11));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    // the rest in FP64: all of it for wide channels, else from the first large change on
    for (; n < end; ++n, next()) {
        uint32_t h[8 * NBW];
        load_h(h);
        const int z = zs[u * M::THREADS];
        double tr = 0.0, ti = 0.0;
#pragma unroll
        for (int i = 0; i < 8 * NBW; ++i) {
            const double hr = fx_lo(h[i]), hi = fx_hi(h[i]), rr = fx_lo(r[i]), ri = fx_hi(r[i]);
            tr = fma(hr, rr, fma(hi, ri, tr));
            ti = fma(hr, ri, fma(-hi, rr, ti));
        }
        tr += __shfl_xor(tr, 16, 64);
        ti += __shfl_xor(ti, 16, 64);
        tr += __shfl_xor(tr, 32, 64);
        ti += __shfl_xor(ti, 32, 64);
        const int dc = change(comp ? ti : tr, z);
        zs[u * M::THREADS] = z + dc;
        const auto both = __builtin_amdgcn_permlane16_swap((unsigned)dc, (unsigned)dc, false, false);
        const double fr = (int)both[0], fi = (int)both[1];
#pragma unroll
        for (int i = 0; i < 8 * NBW; ++i) {
            const uint32_t hx = fx_opaque(h[i]), rx = fx_opaque(r[i]);
            const double hr = fx_lo(hx), hi = fx_hi(hx);
            const double dre = floor(fma(hr, fr, fma(-hi, fi, 1024.0)) * (1.0 / 2048.0));
            const double dim = floor(fma(hr, fi, fma(hi, fr, 1024.0)) * (1.0 / 2048.0));
            r[i] = fx_pack((int)fx_sat16d(fx_lo(rx) - dre), (int)fx_sat16d(fx_hi(rx) - dim));
        }
    }

    // outputs: a lane has its component of its symbol's z; the users dealt over the waves
    // and pairs of lane groups
    if (sym >= ns) return;
    for (int u = (g >> 1) + 2 * wave; u < U; u += 2 * NW) {
        const int z = zs[u * M::THREADS];
        const size_t o = (size_t)v * U + u;
        if (P.z) P.z[2 * o + comp] = (int16_t)z;
        if (P.llr) fx_axis_llrs(P, (float)us[u].p, us[u].g, z, comp, o);
    }
}

template <int NBW, int NW>
static hipError_t launch_fx_tile(const FxParams &p, hipStream_t s)
{
    using M = FxTile<NBW, NW>;
    auto fn = k_fixed_tile<NBW, NW>;
    const size_t lds = M::bytes(p.U);
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    const int tiles = (p.S + 15) / 16;
    const bool vec = p.B % 4 == 0 && reinterpret_cast<uintptr_t>(p.H) % 16 == 0 &&
                     reinterpret_cast<uintptr_t>(p.y) % 16 == 0;
    const int most = (int)groups_per_launch(tiles, M::THREADS);
    for (long w0 = 0; w0 < p.W; w0 += most) {
        FxParams q = p;
        const size_t v0 = (size_t)w0 * p.S;
        q.W = (int)(p.W - w0 < most ? p.W - w0 : most);
        q.H = p.H + (size_t)w0 * p.U * p.B * 2;
        q.y = p.y + v0 * p.B * 2;
        if (p.z) q.z = p.z + v0 * p.U * 2;
        if (p.llr) q.llr = p.llr + v0 * p.U * p.Q;
        hipLaunchKernelGGL(fn, dim3((unsigned)q.W * tiles), dim3(M::THREADS), lds, s, q, tiles, vec);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Channels are staged when the subcarriers a workgroup can touch fit in 32 KB of
// LDS (B = 128, U = 8, S = 14: two subcarriers, 16 KB).
template <int L, int NPL>
static hipError_t launch_fx_t(const FxParams &p, hipStream_t s)
{
    constexpr int G = 256 / L;
    const long nvec = (long)p.W * p.S;
    const dim3 grid((unsigned)((nvec + G - 1) / G));
    const long slots = std::min<long>(G, (G - 1) / p.S + 2);
    const size_t lds = (size_t)slots * p.U * p.B * sizeof(float2);
    if (lds <= 32768)
        hipLaunchKernelGGL((k_forward_fx<L, NPL, true>), grid, dim3(256), lds, s, p);
    else
        hipLaunchKernelGGL((k_forward_fx<L, NPL, false>), grid, dim3(256), 0, s, p);
    return hipGetLastError();
}

// 16 lanes per vector up to B = 128, 32 above: each update is a serial chain (64-bit
// sums across the group, then the narrowing), so with many entries per lane more,
// shorter lanes hide it better (B = 256: 199 -> 154 us per 16,800 vectors at 32
// lanes; B = 64 is faster at 16 lanes, 51 against 63 us).  At B = 128 the columns'
// global-memory round trips made 32 lanes the faster (88 against 84 us); with the
// columns staged in LDS, 16 lanes are (77.5 against 80.1 us, int16 pairs staged).
// At B = 256 32 lanes stay ahead when staged (U = 8, 600 x 14 vectors: 81 against
// 105 us; U = 32, 330 x 14: 229 against 244 us).
//
// The tiles of 16 symbols up to B = 256, where enough of a tile's columns are symbols:
// 4000 subcarriers of 128 x 8, K = 3, tile / lane groups: 94 / 62 us at S = 4, 93 / 89 at
// 6, 98 / 177 at 14.  With fewer symbols also where every SIMD gets at most one wave (1024
// of them), as the chain of a tile's update is the shorter: 1 symbol of 600 x 128 x 8 28 /
// 33 us, of 1200 37 / 33; 2 symbols of 256 subcarriers of 256 x 8 21 / 34, of 600 38 / 35.
static hipError_t launch_fx(const FxParams &p, hipStream_t s)
{
    const int waves = p.B <= 64 ? 1 : p.B <= 128 ? 2 : 4;
    if (p.B <= 256 && (p.S >= 7 || (long)p.W * waves <= 1024) &&
        reinterpret_cast<uintptr_t>(p.y) % 4 == 0) {   // y is read in pairs
        if (p.B <= 32) return launch_fx_tile<1, 1>(p, s);
        if (p.B <= 64) return launch_fx_tile<2, 1>(p, s);
        if (p.B <= 128) return launch_fx_tile<2, 2>(p, s);
        return launch_fx_tile<2, 4>(p, s);
    }
    if (p.B <= 32) return launch_fx_t<16, 2>(p, s);
    if (p.B <= 64) return launch_fx_t<16, 4>(p, s);
    if (p.B <= 128) return launch_fx_t<16, 8>(p, s);
    if (p.B <= 256) return launch_fx_t<32, 8>(p, s);
    if (p.B <= 512) return launch_fx_t<32, 16>(p, s);
    return launch_fx_t<32, 32>(p, s);
}

}  // namespace ocd

extern "C" ocd_status ocd_detect_fixed(const ocd_problem *pb, const int16_t *H, const int16_t *y,
                                       int16_t *z, float *llr, hipStream_t stream)
{
    using namespace ocd;
    ocd_status st = validate(pb);
    if (st != OCD_OK) return st;
    if (!H || !y || (!z && !llr)) return OCD_EINVAL;
    if (pb->mode == OCD_HYBRID) return OCD_EUNSUPPORTED;
    FxParams P;
    P.B = pb->B; P.U = pb->U; P.W = pb->W; P.S = pb->S; P.K = pb->K; P.Q = pb->Q;
    P.box = pb->mode == OCD_BOX;
    P.b = 0;
    while ((1 << P.b) < pb->B) ++P.b;
    const double lam = pb->mode == OCD_MMSE ? (double)pb->N0 / (double)pb->Es : 0.0;
    // alpha = round(lambda 2^22) is an operand of the 36-bit adder beside ||h_u||^2
    const double lam_s = std::floor(lam * 4194304.0 + 0.5);
    if (!(lam_s < 34359738368.0)) return OCD_EINVAL;
    P.lam_q = (long long)lam_s;
    const int M = 1 << (pb->Q / 2);
    const double edge = (double)(M - 1) / std::sqrt(2.0 * (double)(M * M - 1) / 3.0);
    const double beta = pb->beta > 0.f ? (double)pb->beta : edge * std::sqrt((double)pb->Es);
    // c is narrowed to a 16-bit word before the clip, so a bound of 2^15 LSB or
    // more clips nothing: 2^15 stands for all of them
    const double beta_s = std::floor(beta * 2048.0 + 0.5);
    P.beta_fx = beta_s < 32768.0 ? (int)beta_s : 32768;
    if (pb->W == 0) return OCD_OK;
    P.lam = (float)lam;
    P.Es = pb->Es; P.N0 = pb->N0;
    P.sqEs = std::sqrt(pb->Es);
    P.qscale = qam_scale(pb->Q);
    P.H = H; P.y = y; P.z = z; P.llr = llr;
    return launch_fx(P, stream) == hipSuccess ? OCD_OK : OCD_EDEVICE;
}
