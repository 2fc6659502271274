// ocd_gram.h -- Algorithm 1 for a subcarrier whose channel several symbols share,
// with the inner products h_u^H r carried instead of the residual r itself.
//
// Every update of Algorithm 1 reads r only through q_u = h_u^H r, and r changes only
// by h_v Delta_v, so the K U updates can be run on the U numbers q (started from the
// matched filters h_u^H y) and the Gram matrix G = H^H H:
//   Delta = d_u (q_u - lambda z_u), clipped so that z_u + Delta stays in the box,
//   z_u += Delta,  q_v -= G_vu Delta  for every v,
// the iterates of the residual form, update by update.  (d_u (h_u^H r) + p_u z_u with
// p_u = d_u g_u is z_u + d_u (q_u - lambda z_u).)  H and y are then read once, in one
// contraction, instead of twice per update: 4 U^2 B / S + 8 U B + 8 K U^2 operations a
// vector against 16 K U B.
//
// A workgroup is four waves on one subcarrier (and up to 16 symbols of it) or, where there
// are many (gram_waves), a wave on each of four subcarriers.
//   1. The contraction, on the matrix cores.  A row of H or y is 2B floats; Re h^H x is the
//      dot product of two such rows and Im h^H x that of x with the row of j h (-Im, Re
//      pairs).  A lane of the matrix operand holds row l mod 16, and since both operands
//      may permute the summation index alike, its four K steps take the four floats of one
//      16-byte load: the operands go from HBM to registers in the matrix layout, with no
//      staging.  Four waves split the antennas into four segments; one wave takes them in
//      turn with the same sums, so both give the same bits.
//   2. The products and sums are FP64 (v_mfma_f64_16x16x4f64).  The residual form's inner
//      products err with the residual, which shrinks from sweep to sweep; these err once,
//      with ||h|| ||y||, and ill-conditioned channels amplify that.  With FP32 sums of 16, 8
//      or 4 products z errs up to 5.4, 3.1 or 2.1 times as much as in the residual form
//      (users correlated 0.99, 64 x 32), in FP64 0.13 to 0.64 times over 21 shapes and 16
//      kinds of channels (i.i.d., users or antennas correlated 0.5 to 0.999, powers over 20
//      to 60 dB, line of sight), and FP64 costs less than sums of 4: 248 us against 281 for
//      3300 x 14 vectors of 256 x 32, 15.0 against 14.8 for 1200 x 14 of 128 x 8 (sums of 8:
//      226, 13.4).  FP16 storage: see gram_half.
//   3. The four waves' partials meet in LDS; 4 or 16 lanes then own one vector and run its
//      updates in FP64 (full rate on this GPU).  The chain of an update is an FMA, the
//      clip, a DPP broadcast of Delta from its owner and two FMAs; what else it takes is
//      formed once per sweep.
// What bounds it: the latency of that chain and of the loads before it, at the workgroups
// whose registers fit a compute unit, then the FP64 matrix products (64 cycles each: 0.50 of
// the time at 256 x 32, 0.36 at 128 x 8) and the vector issue (0.43, 0.30).  Time of a call against the residual form (two passes over the antennas per
// update): 1200 x 14 vectors of 128 x 8, 3 sweeps, 28.0 -> 14.2 us; 4800 x 14 in FP16 storage
// 65.7 -> 27.9; 3300 x 14 of 256 x 32, box, 5 sweeps 546 -> 239.
#pragma once

#include <type_traits>
#include <utility>

#include "ocd_stage.h"

namespace ocd {

typedef float f32x4_acc __attribute__((ext_vector_type(4)));
typedef double f64x4_acc __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));

constexpr int GRAM_WAVES = 4;
constexpr int GRAM_THREADS = 64 * GRAM_WAVES;
constexpr int GRAM_LD = 18;                  // doubles between columns of a 16 x 16 tile in LDS
constexpr int GRAM_TILE = 16 * GRAM_LD;

// Matrix tiles of a subcarrier with up to UP users.  S8: at most 8 symbols, whose real
// and imaginary products (or, for UP = 8, whose products beside the Gram columns) share
// one tile.
//   UP = 8:  rows are [h; j h], so one product gives Re and Im; tiles G, Q (S8: one)
//   UP = 16: Re G, Im G, then Re Q, Im Q (S8: one)
//   UP = 32: Re, Im of G's blocks 00, 01, 11, then Re, Im of Q's blocks 0, 1 (S8: two)
// SY: the symbols so arranged (SY_8: at most 8), or none (SY_NONE: the Gram matrix alone,
// with the same bits).
enum GramSymbols { SY_16, SY_8, SY_NONE };

template <int UP, GramSymbols SY>
struct GramShape {
    static constexpr bool S8 = SY == SY_8, Y = SY != SY_NONE;
    static constexpr int GT = UP == 8 ? (S8 ? 0 : 1) : UP == 16 ? 2 : 6;
    static constexpr int QT = !Y ? 0 : UP == 8 ? 1 : UP == 16 ? (S8 ? 1 : 2) : (S8 ? 2 : 4);
    static constexpr int T = GT + QT;
    static constexpr int HR = UP == 32 ? 2 : 1;          // channel rows per lane
    static constexpr int PARTS = UP == 32 ? 2 : 4;       // wave partials kept in LDS
};

// Sum over the 16 x 16 tile positions this lane holds, in FP64: column lane mod 16, rows
// first, first + STEP, ..
struct GramAcc {
    f64x4_acc v;
};
template <bool HALF>
struct GramRows {
    static constexpr int STEP = HALF ? 1 : 4;
    __device__ static __forceinline__ int first(int lane) { return (lane >> 4) * (HALF ? 4 : 1); }
};

// Two complex entries of a row as they are stored, loaded without a branch or a use:
// entries past B read the row's last valid ones and are zeroed by gram_pair.
template <bool F16>
struct GramRaw {
    typename std::conditional<F16, u32x2_t, f32x4_t>::type v;
};

template <bool F16, bool VEC>
__device__ __forceinline__ GramRaw<F16> gram_load(const unsigned char *base, unsigned row, int b, int B)
{
    GramRaw<F16> x;
    if constexpr (VEC) {   // B even, aligned rows: the pair is in or out together
        const unsigned off = (row * (unsigned)B + min(b, B - 2)) * cbytes<F16>();
        x.v = *global_ptr(reinterpret_cast<const decltype(x.v) *>(base + off));
    } else {
        const unsigned e = row * (unsigned)B;
        const unsigned o0 = (e + min(b, B - 1)) * cbytes<F16>();
        const unsigned o1 = (e + min(b + 1, B - 1)) * cbytes<F16>();
        if constexpr (F16) {
            x.v.x = *global_ptr(reinterpret_cast<const uint32_t *>(base + o0));
            x.v.y = *global_ptr(reinterpret_cast<const uint32_t *>(base + o1));
        } else {
            const float2 p = global_load2(reinterpret_cast<const float2 *>(base + o0));
            const float2 q = global_load2(reinterpret_cast<const float2 *>(base + o1));
            x.v.x = p.x;
            x.v.y = p.y;
            x.v.z = q.x;
            x.v.w = q.y;
        }
    }
    return x;
}

// The pair as four floats, zero past B (tail: the block is not whole).
template <bool F16>
__device__ __forceinline__ float4 gram_pair(const GramRaw<F16> &x, bool tail, int b, int B)
{
    float4 q;
    if constexpr (F16) {
        const float2 p = half2_to_float2(x.v.x), r = half2_to_float2(x.v.y);
        q = make_float4(p.x, p.y, r.x, r.y);
    } else {
        q = make_float4(x.v.x, x.v.y, x.v.z, x.v.w);
    }
    if (tail) {   // the same for the whole wave
        if (b >= B) q.x = q.y = 0.f;
        if (b + 1 >= B) q.z = q.w = 0.f;
    }
    return q;
}

// Row of j x beside row x: Re h^H x = <h, x> and Im h^H x = <j h, x> = <h, -j x>.
__device__ __forceinline__ float4 times_j(float4 q) { return make_float4(-q.y, q.x, -q.w, q.z); }
__device__ __forceinline__ float4 times_mj(float4 q) { return make_float4(q.y, -q.x, q.w, -q.z); }
__device__ __forceinline__ float4 pick(bool c, float4 a, float4 b)
{
    return make_float4(c ? a.x : b.x, c ? a.y : b.y, c ? a.z : b.z, c ? a.w : b.w);
}
// The same on pairs stored in FP16, (re, im) in a dword.
__device__ __forceinline__ u32x2_t times_j(u32x2_t q)
{
    return u32x2_t{__builtin_amdgcn_alignbit(q.x, q.x, 16) ^ 0x8000u,
                   __builtin_amdgcn_alignbit(q.y, q.y, 16) ^ 0x8000u};
}
__device__ __forceinline__ u32x2_t times_mj(u32x2_t q)
{
    return u32x2_t{__builtin_amdgcn_alignbit(q.x, q.x, 16) ^ 0x80000000u,
                   __builtin_amdgcn_alignbit(q.y, q.y, 16) ^ 0x80000000u};
}
__device__ __forceinline__ u32x2_t pick(bool c, u32x2_t a, u32x2_t b)
{
    return u32x2_t{c ? a.x : b.x, c ? a.y : b.y};
}

// Operands of one 8-antenna block: this lane's channel rows and its symbol row.
template <int HR, bool F16>
struct GramBlock {
    GramRaw<F16> h[HR], y;
};

template <int UP, GramSymbols SY, bool F16, bool VEC>
__device__ __forceinline__ void gram_load_block(const Params &P, const unsigned char *hb,
                                                const unsigned char *yb, int blk, int ns,
                                                GramBlock<GramShape<UP, SY>::HR, F16> &x)
{
    const int lane = threadIdx.x & 63, i = lane & 15, b = blk * 8 + (lane >> 4) * 2;
    const int U = P.U, B = P.B;
    // rows past the users and symbols repeat a valid one; their products are never read
    const int hi = UP == 8 ? i & 7 : i;
    x.h[0] = gram_load<F16, VEC>(hb, min(hi, U - 1), b, B);
    if constexpr (UP == 32) x.h[1] = gram_load<F16, VEC>(hb, min(16 + i, U - 1), b, B);
    if constexpr (SY != SY_NONE)
        x.y = gram_load<F16, VEC>(yb, min(SY == SY_8 ? i & 7 : i, ns - 1), b, B);
}

// ||h||^2 of a lane's channel rows in the summation order of k_preprocess, whose lane l of
// 16 sums the entries l, l + 16, ... : the entries of block blk that a lane holds belong
// to l = 8 (blk mod 2) + 2 (lane / 16) and the next one.
template <int HR>
struct GramNorm {
    float v[HR][2][2];

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int r = 0; r < HR; ++r) v[r][0][0] = v[r][0][1] = v[r][1][0] = v[r][1][1] = 0.f;
    }
    __device__ __forceinline__ void add(int r, int odd, const float4 &h)   // odd: wave-uniform
    {
        if (odd) {
            v[r][1][0] = fmaf(h.x, h.x, fmaf(h.y, h.y, v[r][1][0]));
            v[r][1][1] = fmaf(h.z, h.z, fmaf(h.w, h.w, v[r][1][1]));
        } else {
            v[r][0][0] = fmaf(h.x, h.x, fmaf(h.y, h.y, v[r][0][0]));
            v[r][0][1] = fmaf(h.z, h.z, fmaf(h.w, h.w, v[r][0][1]));
        }
    }
    // the levels of group_sum<16>: l ^ 1 here, l ^ 2 and the other half of 8 in the lanes
    // 16 and 32 away, the other 8 here
    __device__ __forceinline__ float sum(int r) const
    {
        float s[2];
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            s[o] = v[r][o][0] + v[r][o][1];
            s[o] += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(s[o]), 0x401F));
            const int src = (static_cast<int>(__lane_id()) ^ 32) << 2;
            s[o] += __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(s[o])));
        }
        return s[0] + s[1];
    }
};

__device__ __forceinline__ float comp(const float4 &q, int c)
{
    return c == 0 ? q.x : c == 1 ? q.y : c == 2 ? q.z : q.w;
}

// The products of one block into every tile: four K steps in FP64 or (HALF, FP16 storage)
// two FP32 sums of eight products (v_mfma_f32_16x16x16_f16, the first and the second entry of
// every pair), added in FP64.  NORM: the lane's squares of its channel rows as well (see
// GramNorm).
template <int UP, GramSymbols SY, bool F16, bool HALF, bool NORM>
__device__ __forceinline__ void gram_block(const GramBlock<GramShape<UP, SY>::HR, F16> &raw,
                                           int blk, int B, GramAcc (&acc)[GramShape<UP, SY>::T],
                                           GramNorm<GramShape<UP, SY>::HR> &gsq)
{
    static_assert(F16 || !HALF, "FP16 operands from FP16 storage");
    using Sh = GramShape<UP, SY>;
    constexpr bool S8 = Sh::S8;
    const int b = blk * 8 + ((threadIdx.x >> 4) & 3) * 2;
    const bool tail = blk * 8 + 8 > B;
    using Op = typename std::conditional<HALF, u32x2_t, float4>::type;
    auto operand = [&](const GramRaw<F16> &q) -> Op {
        if constexpr (HALF) {
            u32x2_t v = q.v;
            if (tail) {   // the same for the whole wave
                if (b >= B) v.x = 0;
                if (b + 1 >= B) v.y = 0;
            }
            return v;
        } else {
            return gram_pair<F16>(q, tail, b, B);
        }
    };
    struct {
        Op h[Sh::HR], y;
    } x;
#pragma unroll
    for (int r = 0; r < Sh::HR; ++r) x.h[r] = operand(raw.h[r]);
    if constexpr (Sh::Y) x.y = operand(raw.y);
    else x.y = Op{};
    if constexpr (NORM) {
#pragma unroll
        for (int r = 0; r < Sh::HR; ++r) gsq.add(r, blk & 1, gram_pair<F16>(raw.h[r], tail, b, B));
    }
    const bool low = (threadIdx.x & 15) < 8;
    Op a[2 * Sh::HR];   // rows h and j h
    Op bq;              // the symbols' columns
    if constexpr (UP == 8) {
        a[0] = a[1] = pick(low, x.h[0], times_j(x.h[0]));
        bq = S8 ? pick(low, x.h[0], x.y) : x.y;
    } else {
#pragma unroll
        for (int r = 0; r < Sh::HR; ++r) {
            a[2 * r] = x.h[r];
            a[2 * r + 1] = times_j(x.h[r]);
        }
        bq = S8 ? pick(low, x.y, times_mj(x.y)) : x.y;
    }
    const f32x4_acc zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < (HALF ? 2 : 4); ++c) {
        f32x4_acc d[HALF ? Sh::T : 1];
        auto mm = [&](int t, const Op &p, const Op &q) {
            if constexpr (HALF) {
                auto one = [&](const u32x2_t &x) {   // of both operands: 0 times inf is not 0
                    return __builtin_bit_cast(f16x4_t, c == 0 ? u32x2_t{x.x, 0u} : u32x2_t{x.y, 0u});
                };
                d[t] = __builtin_amdgcn_mfma_f32_16x16x16f16(one(p), one(q), zero, 0, 0, 0);
            } else {
                acc[t].v = __builtin_amdgcn_mfma_f64_16x16x4f64((double)comp(p, c),
                                                                (double)comp(q, c), acc[t].v, 0, 0, 0);
            }
        };
        if constexpr (UP == 8) {
            if constexpr (!S8) mm(0, a[0], x.h[0]);
            if constexpr (Sh::Y) mm(Sh::T - 1, a[0], bq);
        } else if constexpr (UP == 16) {
            mm(0, a[0], x.h[0]);
            mm(1, a[1], x.h[0]);
            if constexpr (Sh::Y) mm(2, a[0], bq);
            if constexpr (Sh::Y && !S8) mm(3, a[1], bq);
        } else {
            mm(0, a[0], x.h[0]);
            mm(1, a[1], x.h[0]);
            mm(2, a[0], x.h[1]);
            mm(3, a[1], x.h[1]);
            mm(4, a[2], x.h[1]);
            mm(5, a[3], x.h[1]);
            if constexpr (Sh::Y) mm(6, a[0], bq);
            if constexpr (S8) {
                mm(7, a[2], bq);
            } else if constexpr (Sh::Y) {
                mm(7, a[1], bq);
                mm(8, a[2], bq);
                mm(9, a[3], bq);
            }
        }
        if constexpr (HALF) {
#pragma unroll
            for (int t = 0; t < Sh::T; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[t].v[r] += (double)d[t][r];
        }
    }
}

// The antennas are cut into four segments of whole blocks of 8, each summed by itself and
// the segments then added in order: one wave per segment (NW = 4) or one wave for all of
// them (NW = 1) give the same bits.  The next blocks' loads are in flight while the
// current ones multiply; `between` runs when the first are out.
template <int UP, GramSymbols SY, bool F16, bool VEC, bool HALF, int NW, typename Between>
__device__ __forceinline__ void gram_contract(const Params &P, const unsigned char *hb,
                                              const unsigned char *yb, int ns,
                                              GramAcc (&acc)[GramShape<UP, SY>::T],
                                              GramNorm<GramShape<UP, SY>::HR> &gsq,
                                              Between &&between)
{
    using Sh = GramShape<UP, SY>;
    constexpr int T = Sh::T;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nblk = (P.B + 7) >> 3;
    const int m1 = nblk / 4, m2 = 2 * nblk / 4, m3 = 3 * nblk / 4;   // ends of segments
    const int b0 = NW == 4 ? wave * nblk / 4 : 0, b1 = NW == 4 ? (wave + 1) * nblk / 4 : nblk;
    const int last = max(b1 - 1, 0);
    GramAcc tot[NW == 1 ? T : 1];
    if constexpr (NW == 1) {
#pragma unroll
        for (int t = 0; t < T; ++t) tot[t] = acc[t];
    }
    // two blocks in turn, each loaded again as soon as it is multiplied, with no copy or
    // branch, either of which would wait for the loads: past its end a wave reads its last
    // block again.  (Four blocks in flight take registers that are worth more as waves: 1.08
    // times as long at 256 x 32, 1.17 at 128 x 16, measured with FP32 products.)  The barrier
    // after the last pass waits for that pass's loads: four waves on few users, whose passes
    // are few, peel it (1200 x 14 vectors of 128 x 8: 15.0 us without, 14.9 with, in FP16
    // storage 13.3 and 11.8; 700 x 7 of 128 x 4 9.0 and 8.5); elsewhere it changes nothing and
    // is a second copy of the products
    constexpr bool PEEL = NW == 4 && UP == 8;
    GramBlock<Sh::HR, F16> x0, x1;
    auto load = [&](GramBlock<Sh::HR, F16> &x, int blk) {
        gram_load_block<UP, SY, F16, VEC>(P, hb, yb, min(blk, last), ns, x);
    };
    auto multiply = [&](const GramBlock<Sh::HR, F16> &x, int e) {
        if (e >= b1) return;
        gram_block<UP, SY, F16, HALF, NW == 1>(x, e, P.B, acc, gsq);
        if (NW == 1 && ((e + 1 == m1) | (e + 1 == m2) | (e + 1 == m3))) {
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    tot[NW == 1 ? t : 0].v[r] += acc[t].v[r];
                    acc[t].v[r] = 0.0;
                }
        }
    };
    load(x0, b0);
    load(x1, b0 + 1);
    between();
    int blk = b0;
    for (; (PEEL ? blk + 2 : blk) < b1; blk += 2) {
        multiply(x0, blk);
        load(x0, blk + 2);
        multiply(x1, blk + 1);
        load(x1, blk + 3);
    }
    if constexpr (PEEL) {
        multiply(x0, blk);
        multiply(x1, blk + 1);
    }
    if constexpr (NW == 1) {
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[t].v[r] = tot[t].v[r] + acc[t].v[r];
    }
}

// LDS position of tile t, column c, row r of a wave partial.
template <int T>
__device__ __forceinline__ int gram_at(int part, int t, int c, int r)
{
    return (part * T + t) * GRAM_TILE + c * GRAM_LD + r;
}

// LDS of a workgroup.  NW = 4 (four waves on one subcarrier): the waves' partial tiles,
// then, in their place, the Gram matrix G[v][u] = h_u^H h_v (column v contiguous) and the
// matched filters Q[s][u], (re, im).  NW = 1 (a subcarrier per wave): G and Q of each.
template <int UP, GramSymbols SY, int NW>
struct GramLds {
    using Sh = GramShape<UP, SY>;
    static constexpr int SG = GRAM_WAVES / NW;   // subcarriers of a workgroup
    static constexpr int PART = NW == 4 ? Sh::PARTS * Sh::T * GRAM_TILE : 0;
    static constexpr int G = 0, Q = 2 * UP * UP;
    // + 2: the waves that sweep several subcarriers read the same column of each, 4 or 16
    // lanes of 64 bytes apart: 16 bytes more between subcarriers keep them off each
    // other's banks
    static constexpr int SUMS = Q + (SY == SY_8 ? 8 : SY == SY_16 ? 16 : 0) * 2 * UP + 2;
    static constexpr int DOUBLES = PART > SG * SUMS ? PART : SG * SUMS;
};

// Per user: ||h_u||^2 and the soft output's constants of llr_coef, L_b = c D_b(a z_u),
// formed in FP64 (t = a z is of the size of the constellation's levels, and the metrics
// D_b take differences of it: every rounding of a is one of t).
struct GramUser {
    double a;
    float c, g;
};

__device__ __forceinline__ GramUser gram_user(const Params &P, float g, float pK, float lamK)
{
    const double mu = lamK > 0.f ? (double)pK : 1.0;
    const double rho = lamK > 0.f ? (double)g / lamK : (double)g * P.Es / P.N0;
    const bool on = rho > 0.0 && mu > 0.0;   // else a zero column: all of its LLRs are zero
    return {on ? P.llr_a / mu : 0.0, on ? (float)(rho * P.llr_c) : 0.f, g};
}

// d_u^-1 of user u of subcarrier w in sweep k, and p_u: the given values, or from
// g = ||h_u||^2 as k_preprocess forms them.
__device__ __forceinline__ float gram_dinv(const Params &P, long w, int k, int u, float g,
                                           float lam, float *p)
{
    if (P.dinv_in) {
        const int Kt = P.per_sweep ? P.K : 1;
        const long o = (w * Kt + (P.per_sweep ? k : 0)) * P.U + u;
        *p = global_ptr(P.p_in)[o];
        return global_ptr(P.dinv_in)[o];
    }
    const float den = g + lam;
    const float di = den > 0.f ? 1.0f / den : 0.f;
    *p = di * g;
    return di;
}

// Contraction of subcarrier w with symbols s0 .. s0 + ns - 1 by this wave (NW = 1; lds, us
// its own) or workgroup (NW = 4), and the users' constants, ||h_u||^2 in the summation
// order of k_preprocess, so that d^-1 and p have its bits.  Ends with a workgroup barrier.
template <int UP, GramSymbols SY, bool F16, bool VEC, bool HALF, int NW>
__device__ __forceinline__ void gram_front(const Params &P, long w, int s0, int ns, double *lds,
                                           GramUser *us)
{
    using Sh = GramShape<UP, SY>;
    constexpr int T = Sh::T;
    const int U = P.U, B = P.B;
    const unsigned char *hb =
        static_cast<const unsigned char *>(P.H) + (size_t)w * U * B * cbytes<F16>();
    const unsigned char *yb =
        static_cast<const unsigned char *>(P.y) + ((size_t)w * P.S + s0) * B * cbytes<F16>();
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    GramAcc acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[t].v[r] = 0.0;
    auto finish_user = [&](int u, float g) {
        const float lamK = P.lambda ? global_ptr(P.lambda)[P.K - 1] : P.lam_default;
        float pK;
        gram_dinv(P, w, P.K - 1, u, g, lamK, &pK);
        us[u] = gram_user(P, g, pK, lamK);
    };
    GramNorm<Sh::HR> gsq;
    gsq.clear();
    if constexpr (NW == 1) {
        gram_contract<UP, SY, F16, VEC, HALF, NW>(P, hb, yb, ns, acc, gsq, [] {});
#pragma unroll
        for (int r = 0; r < Sh::HR; ++r) {
            const float g = gsq.sum(r);   // of row lane mod 16
            const int u = lane + 16 * r;
            if (lane < (UP < 16 ? UP : 16) && u < U)
                finish_user(u, P.g_in ? global_ptr(P.g_in)[w * U + u] : g);
        }
    } else {
        // 16 lanes per column, lane l summing entries l, l + 16, ...; the first 128
        // antennas of 16 columns are loaded ahead of the operands (the same lines)
        const int u0 = tid >> 4, l16 = tid & 15;
        auto entry = [&](int u, int b) -> float2 {
            const unsigned e = (unsigned)min(u, U - 1) * B + min(b, B - 1);
            if constexpr (!F16) return global_load2(reinterpret_cast<const float2 *>(hb) + e);
            else return half2_to_float2(global_ptr(reinterpret_cast<const uint32_t *>(hb))[e]);
        };
        auto square = [&](float2 v, int b, float s) {
            return b < B ? fmaf(v.x, v.x, fmaf(v.y, v.y, s)) : s;
        };
        const bool own_g = P.g_in == nullptr, first_g = own_g && (wave * 4 < U);
        float2 hg[8];
        if (first_g) {
#pragma unroll
            for (int i = 0; i < 8; ++i) hg[i] = entry(u0, l16 + 16 * i);
        }
        float s0g = 0.f;
        gram_contract<UP, SY, F16, VEC, HALF, NW>(P, hb, yb, ns, acc, gsq, [&] {
            if (first_g) {
#pragma unroll
                for (int i = 0; i < 8; ++i) s0g = square(hg[i], l16 + 16 * i, s0g);
            }
        });
        for (int u = u0; u < U; u += 16) {
            float s = 0.f;
            if (own_g) {
                int b0 = 0;
                if (u == u0) {
                    s = s0g;
                    b0 = 128;
                }
                for (; b0 < B; b0 += 128) {
                    float2 x[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) x[i] = entry(u, b0 + l16 + 16 * i);
#pragma unroll
                    for (int i = 0; i < 8; ++i) s = square(x[i], b0 + l16 + 16 * i, s);
                }
                s = group_sum<16>(s);
            } else {
                s = global_ptr(P.g_in)[w * U + u];
            }
            if (l16 == 0) finish_user(u, s);
        }
    }

    double *G = lds + GramLds<UP, SY, NW>::G, *Q = lds + GramLds<UP, SY, NW>::Q;
    auto put = [&](double *m, int v, int u, int im, double x) { m[2 * (v * UP + u) + im] = x; };
    auto place = [&](int c, int r, const double (&sum)[T]) {   // position (c, r) of every tile
        if constexpr (UP == 8) {
            if constexpr (Sh::S8) {
                put(c < 8 ? G : Q, c & 7, r & 7, r >> 3, sum[0]);
            } else {
                if (c < 8) put(G, c, r & 7, r >> 3, sum[0]);
                if constexpr (Sh::Y) put(Q, c, r & 7, r >> 3, sum[1]);
            }
        } else {
#pragma unroll
            for (int im = 0; im < 2; ++im) {
                put(G, c, r, im, sum[im]);
                if constexpr (UP == 32) {
                    put(G, 16 + c, r, im, sum[2 + im]);
                    put(G, r, 16 + c, im, im ? -sum[3] : sum[2]);   // block 10 = block 01^H
                    put(G, 16 + c, 16 + r, im, sum[4 + im]);
                }
            }
#pragma unroll
            for (int q = 0; q < Sh::QT; ++q) {
                if constexpr (Sh::S8) put(Q, c & 7, r + 16 * q, c >> 3, sum[Sh::GT + q]);
                else put(Q, c, r + 16 * (q >> 1), q & 1, sum[Sh::GT + q]);
            }
        }
    };
    using Rows = GramRows<HALF>;
    const int col = lane & 15, row = Rows::first(lane);
    if constexpr (NW == 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double sum[T];
#pragma unroll
            for (int t = 0; t < T; ++t) sum[t] = acc[t].v[r];
            place(col, row + Rows::STEP * r, sum);
        }
        __syncthreads();
        return;
    }
    auto store = [&](int p) {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            double *d = lds + gram_at<T>(p, t, col, row);
#pragma unroll
            for (int r = 0; r < 4; ++r) d[Rows::STEP * r] = acc[t].v[r];
        }
    };
    if constexpr (Sh::PARTS == 2) {   // waves 2 and 3 hand theirs to 0 and 1 first
        if (wave >= 2) store(wave - 2);
        __syncthreads();
        if (wave < 2) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const double *d = lds + gram_at<T>(wave, t, col, row);
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[t].v[r] += d[Rows::STEP * r];
            }
            store(wave);
        }
    } else {
        store(wave);
    }
    __syncthreads();
    // thread (c, r) sums position (c, r) of every tile over the waves, in wave order
    const int c = tid >> 4, r = tid & 15;
    double sum[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        sum[t] = lds[gram_at<T>(0, t, c, r)];
#pragma unroll
        for (int p = 1; p < Sh::PARTS; ++p) sum[t] += lds[gram_at<T>(p, t, c, r)];
    }
    __syncthreads();
    place(c, r, sum);
    __syncthreads();
}

// The value of lane N of every aligned group of L = 4, 8 or 16 lanes: quad_perm [N,N,N,N],
// or row_newbcast, the one DPP move that takes both halves of a double at once.
template <int L, int N>
__device__ __forceinline__ double group_bcast(double x)
{
    if constexpr (L == 4) {
        const long long b = __double_as_longlong(x);
        const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)b, 0x55 * N, 0xF, 0xF, true);
        const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x55 * N, 0xF, 0xF, true);
        return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
    } else {
        double y = __builtin_amdgcn_mov_dpp(x, 0x150 + N, 0xF, 0xF, true);
        if constexpr (L == 8) y = __builtin_amdgcn_update_dpp(y, x, 0x158 + N, 0xF, 0xC, false);
        return y;
    }
}

template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// f(std::integral_constant<int, 0>) .. f(... N - 1): DPP controls are immediates.
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// d_u^-1 of this lane's users i R .. i R + R - 1 in sweep k, and their regulariser.
template <int R>
__device__ __forceinline__ double gram_coefs(const Params &P, long w, int k, int i,
                                             const GramUser *us, double (&d)[R])
{
    const float lam = P.lambda ? global_ptr(P.lambda)[k] : P.lam_default;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int u = i * R + r, uu = min(u, P.U - 1);
        float p;
        const float di = gram_dinv(P, w, k, uu, us[uu].g, lam, &p);
        d[r] = u < P.U ? di : 0.f;   // users past U: d = 0, never updated
    }
    return lam;
}

// p_u - 1 in sweep k: -d lambda, or -1 with d = 0, where z_u goes to p_u z_u = 0; with
// given d^-1 and p that are not those of g and lambda, by p itself.
__device__ __forceinline__ double gram_pull(const Params &P, long w, int k, int u, float g,
                                            double d, double lam)
{
    if (P.p_in) {
        float p;
        const float di = gram_dinv(P, w, k, u, g, (float)lam, &p), den = g + (float)lam;
        if (!(den > 0.f && di == 1.0f / den && p == di * g)) return (double)p - 1.0;
    }
    return d > 0.0 ? -d * lam : -1.0;
}

// The K sweeps of one vector on L lanes, lane i owning users i R .. i R + R - 1 (R =
// UP / L): G the Gram matrix, q this lane's matched filters; sweep_done(k) with z in the
// lane's z after every sweep.  z_u changes once per sweep, at its own update, so what
// Delta_u = d q_u - (d lambda) z_u needs of it, and the bounds [-beta - z_u, beta - z_u]
// of Delta_u in the box, are formed before the sweep: the chain from one update to the
// next is one FMA, the clip, the broadcast and two FMAs.
template <int UP, bool BOX, int L, typename Done>
__device__ __forceinline__ void gram_run(const Params &P, long w, int i, const double2 *G,
                                         const GramUser *us, double2 (&q)[UP / L],
                                         double2 (&z)[UP / L], Done &&sweep_done)
{
    constexpr int R = UP / L;
    const int U = P.U, K = P.K;
    const double beta = P.beta;
    G += i * R;
    double d[R], lam = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) z[r] = make_double2(0.0, 0.0);
    if (!P.per_sweep) lam = gram_coefs<R>(P, w, 0, i, us, d);
    for (int k = 0; k < K; ++k) {
        if (P.per_sweep) lam = gram_coefs<R>(P, w, k, i, us, d);
        double2 t[R], lo[BOX ? R : 1], hi[BOX ? R : 1];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int u = min(i * R + r, U - 1);
            const double e = gram_pull(P, w, k, u, us[u].g, d[r], lam);
            t[r] = make_double2(e * z[r].x, e * z[r].y);
            if constexpr (BOX) {
                lo[r] = make_double2(-beta - z[r].x, -beta - z[r].y);
                hi[r] = make_double2(beta - z[r].x, beta - z[r].y);
            }
        }
        static_for<UP / 4>([&](auto cc) {   // four updates at a time (users past U change nothing)
            constexpr int c = decltype(cc)::value;
            if (4 * c < U) {
                static_for<4>([&](auto uc) {
                    constexpr int u = 4 * c + decltype(uc)::value, o = u / R, n = u % R;
                    double cr = fma(d[n], q[n].x, t[n].x), ci = fma(d[n], q[n].y, t[n].y);
                    if constexpr (BOX) {
                        cr = fmin(fmax(cr, lo[n].x), hi[n].x);
                        ci = fmin(fmax(ci, lo[n].y), hi[n].y);
                    }
                    const double dr = group_bcast<L, o>(cr), di = group_bcast<L, o>(ci);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const double2 a = G[u * UP + r];
                        q[r].x = fma(-a.x, dr, fma(a.y, di, q[r].x));
                        q[r].y = fma(-a.x, di, fma(-a.y, dr, q[r].y));
                    }
                    const double own = i == o ? 1.0 : 0.0;   // the owner's z
                    z[n].x = fma(own, cr, z[n].x);
                    z[n].y = fma(own, ci, z[n].y);
                });
            }
        });
        sweep_done(k);
    }
}

// The LLRs of one user, the Q / 2 of each axis (llr: the user's Q values).
template <typename Dst>
__device__ __forceinline__ void gram_llrs(const Params &P, double2 z, const GramUser &us, Dst llr)
{
    const double ua = us.a;
    const float uc = us.c, tr = (float)(z.x * ua), ti = (float)(z.y * ua);
    const int half = P.Q >> 1;
    if (half == 3) {
        axis_llrs<3>(tr, uc, llr);
        axis_llrs<3>(ti, uc, llr + 3);
    } else if (half == 2) {
        axis_llrs<2>(tr, uc, llr);
        axis_llrs<2>(ti, uc, llr + 2);
    } else {
        axis_llrs<1>(tr, uc, llr);
        axis_llrs<1>(ti, uc, llr + 1);
    }
}

// Lanes per vector: with 4, one wave holds 16 vectors and an update costs the fewest
// instructions; 16 (one vector per DPP row) where few vectors or many users would leave
// one wave with a long chain.
template <int UP, GramSymbols SY, int NW>
constexpr int gram_lanes()
{
    return UP == 32 || (UP == 16 && SY == SY_8 && NW == 4) ? 16 : 4;
}

// The vector of a lane group after gram_front: which of the workgroup's SG subcarriers
// (from w0 on; those past W repeat the last), which symbol of the tile, and whether there
// is such a vector.  With a subcarrier per wave, tiles of up to 4 or 8 symbols put the
// vectors of four or two subcarriers into one wave.
template <int L, int NW>
struct GramVector {
    int i, sub, s;
    bool active, wave_idle;
    long w;

    __device__ __forceinline__ GramVector(const Params &P, long w0, int ns)
    {
        constexpr int SG = GRAM_WAVES / NW;
        const int slot = threadIdx.x / L;
        i = threadIdx.x % L;
        const int sh = NW == 4 ? 8 : ns <= 4 ? 2 : ns <= 8 ? 3 : 4;
        sub = slot >> sh;
        s = slot - (sub << sh);
        active = sub < SG && s < ns && w0 + sub < P.W;
        // idle when the wave's first vector is past the end (its others follow it)
        wave_idle = __builtin_amdgcn_readfirstlane(
            NW == 4 ? s >= ns : sub >= SG || w0 + sub >= P.W);
        sub = min(sub, SG - 1);
        s = min(s, ns - 1);
        w = min(w0 + sub, (long)P.W - 1);
    }
};

// The K sweeps and the outputs of the workgroup's vectors after gram_front.  Waves
// without a vector return at once.
template <int UP, GramSymbols SY, bool BOX, int NW>
__device__ __forceinline__ void gram_sweeps(const Params &P, long w0, int s0, int ns,
                                            const double *lds, const GramUser *us)
{
    constexpr int L = gram_lanes<UP, SY, NW>(), R = UP / L;
    using M = GramLds<UP, SY, NW>;
    const int U = P.U, K = P.K;
    const GramVector<L, NW> x(P, w0, ns);
    if (x.wave_idle) return;
    const long v = x.w * P.S + s0 + x.s;
    const double *m = lds + x.sub * M::SUMS;
    const double2 *G = reinterpret_cast<const double2 *>(m + M::G);
    const double2 *Q = reinterpret_cast<const double2 *>(m + M::Q) + x.s * UP + x.i * R;
    us += x.sub * UP;
    double2 q[R], z[R];
#pragma unroll
    for (int r = 0; r < R; ++r) q[r] = Q[r];
    gram_run<UP, BOX, L>(P, x.w, x.i, G, us, q, z, [&](int k) {
        if (P.z_hist && x.active) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (x.i * R + r < U)
                    global_store2(P.z_hist + (v * K + k) * U + x.i * R + r,
                                  make_float2((float)z[r].x, (float)z[r].y));
        }
    });
    if (!x.active) return;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int u = x.i * R + r;
        if (u >= U) continue;
        if (P.z) global_store2(P.z + v * U + u, make_float2((float)z[r].x, (float)z[r].y));
        if (P.llr) gram_llrs(P, z[r], us[u], global_ptr(P.llr) + (v * U + u) * P.Q);
    }
}

// Whether the contraction of FP16 storage takes FP16 operands (exact products, FP32 sums of
// eight): where z then errs no more than in the residual form on any of the channels above
// (16 antennas a user, up to 8 users and 16 sweeps: 0.7 to 0.99 times at the worst; 128 x 8
// at 32 sweeps 1.03, 256 x 16 at 16 1.11, 128 x 16 1.09).  4800 x 14 vectors of 128 x 8 30 us
// against 40 in FP64, 1200 x 14 11.8 against 14.8.
__host__ __device__ inline bool gram_half(int B, int U, int K)
{
    return U <= 8 && B >= 16 * U && K <= 16;
}

// f(VEC, HALF) as integral constants, one return type.  VEC: rows of even length, aligned.
template <int UP, bool F16, typename F>
__host__ __device__ __forceinline__ auto gram_dispatch(const Params &P, F &&f)
{
    using std::false_type;
    using std::true_type;
    if constexpr (F16 && UP == 8) {
        if (gram_half(P.B, P.U, P.K))
            return P.vec_ok ? f(true_type{}, true_type{}) : f(false_type{}, true_type{});
    }
    return P.vec_ok ? f(true_type{}, false_type{}) : f(false_type{}, false_type{});
}

// This wave's subcarrier of a workgroup whose first is w0.
template <int NW>
__device__ __forceinline__ long gram_subcarrier(const Params &P, long w0)
{
    const int sub = NW == 4 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    return min(w0 + sub, (long)P.W - 1);
}

// One tile: symbols s0 .. s0 + ns - 1 of the workgroup's subcarriers, from w0 on.
template <int UP, GramSymbols SY, bool F16, bool BOX, bool VEC, bool HALF, int NW>
__device__ __forceinline__ void gram_tile(const Params &P, long w0, int s0, int ns, double *lds,
                                          GramUser *us)
{
    using M = GramLds<UP, SY, NW>;
    const int sub = NW == 4 ? 0 : threadIdx.x >> 6;
    gram_front<UP, SY, F16, VEC, HALF, NW>(P, gram_subcarrier<NW>(P, w0), s0, ns,
                                         lds + sub * M::SUMS, us + sub * UP);
    gram_sweeps<UP, SY, BOX, NW>(P, w0, s0, ns, lds, us);
}

// Waves per subcarrier: one where there are enough subcarriers (and tiles of 16 symbols of
// them) to keep the GPU busy (no partial sums to exchange, and the set-up once per
// subcarrier), four below, where the length of a workgroup's chain counts.  The line moves
// down with the antennas, whose matrix products the four waves share, and for more than 8
// users and symbols, whose sweeps keep one wave of the four busy for long.  Time with one wave over
// time with four (K = 2, 4):
//   32 x 8:   1.00 at 400, 0.94 at 520 (S <= 8); 1.12, 1.03, 0.99 at 700 (S > 8)
//   64 x 8:   1.05-1.18 at 1030, 0.99-1.08 at 1300, 0.91-1.00 at 1600
//   128 x 8:  1.03-1.14 at 2100, 0.84-0.94 at 3000;  128 x 16, S <= 8: 1.10, 0.89
//   128 x 16, S > 8: 1.14 at 700, 0.94 at 850;  256 x 16: 1.15 at 1030, 0.93 at 1600
// Above 16 users the tiles' FP64 sums of a whole subcarrier do not fit one wave's registers.
__host__ __device__ inline int gram_waves(int B, int U, int S, long subcarrier_tiles)
{
    if (U > 16) return 4;
    const long line = U > 8 && S > 8 ? (B <= 128 ? 800 : 1500)
                      : U <= 8 && B <= 32 ? 600 : B <= 64 ? 1280 : 2500;
    return subcarrier_tiles >= line ? 1 : 4;
}

}  // namespace ocd
