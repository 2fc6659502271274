// ocd_gram_grad.h -- the adjoint of the Gram form (ocd_gram.h) and the training step in
// it: Algorithm 1 and the soft output, the loss, and the reverse sweeps, for the
// subcarriers whose channel several symbols share.
//
// The reverse of update (k, u) reads r_bar only through h_u^H r_bar and adds h_u a to it
// (a = d_u^-1 c_bar), so, as in the forward sweeps, the U numbers w_u = h_u^H r_bar are
// kept instead: w_v += G_vu a.  y_bar = r_bar = sum_u h_u A_u with A_u the sum of u's
// a over the sweeps: one pass over the channel at the end in place of two per update.
// z after every sweep is rounded to FP32 before the reverse sweeps read it, as the history
// that a detection writes is, so that the training step and the adjoint of a detection
// give the same bits of dy.
//
// A workgroup takes tiles blockIdx, blockIdx + grid, ... (a subcarrier and up to tsyms of
// its symbols each) and keeps its partial sums of dlambda_k, dbeta and the loss in LDS
// until the end.
#pragma once

#include "ocd_adjoint.h"
#include "ocd_gram.h"

namespace ocd {

// Whether one wave takes a subcarrier (see gram_waves): from two tiles a compute unit on, or
// where four waves share long sweeps or contractions, from three or four.  Time with one
// wave over time with four, K = 4, at 520 / 700 / 1000 subcarriers:
//   adjoint         128 x 4, S = 8: 0.96 / 0.90 / 0.79;   64 x 8, S = 14: 1.09 / 1.00 / 0.88;
//                   128 x 16, S = 4: 0.63 / 0.60 / 0.59;  256 x 16, S = 14: 1.06 / 1.01 / 0.94
//   training step   32 x 8, S = 8: 0.90 / 0.84 / 0.75;    64 x 8, S = 14: 1.15 / 1.08 / 0.96;
//                   128 x 16, S = 4: 1.29 / 1.23 / 1.08
template <bool TRAIN>
bool grad_one_wave(const Params &p)
{
    const long tiles = (long)p.W * ((p.S + 15) / 16);
    if (p.U <= 8) return tiles > (p.S <= 8 ? 512 : 768);
    if (p.S <= 8) return tiles > (TRAIN ? 1023 : 512);
    return tiles > (TRAIN || p.B <= 128 ? 512 : 768);
}

// Dynamic LDS of a launch: the contraction, the users' constants, A, the partial sums and
// (training step) z after every sweep, for SG subcarriers of up to tsyms symbols.
template <int UP, GramSymbols SY, bool TRAIN, int NW>
struct GradLds {
    using M = GramLds<UP, SY, NW>;
    static constexpr int SG = M::SG;
    static constexpr size_t US = (size_t)M::DOUBLES * 8;
    static constexpr size_t A = US + SG * UP * sizeof(GramUser);
    __host__ __device__ static size_t part(int tsyms) { return A + (size_t)SG * tsyms * UP * 8; }
    __host__ __device__ static size_t zh(int tsyms, int K)
    {
        return part(tsyms) + (size_t)(K + 2) * GRAM_WAVES * 8;
    }
    __host__ __device__ static size_t bytes(int tsyms, int K, int U)
    {
        return zh(tsyms, K) + (TRAIN ? (size_t)SG * tsyms * K * U * 8 : 0);
    }
};

// dLoss/dz of one user (z after the last sweep) through the soft output, and its
// contribution to dLoss/dlambda_K.  In the units of gram_llrs an LLR is c D_b(t), t = a z
// and D_b(t) = (t - l0)^2 - (t - l1)^2 for the nearest levels l0, l1 with the bit 0 and 1,
// so both derivatives are sums over the bits of dLoss/dL_b times l1 - l0 and D_b.  The sums
// are in FP64: what lambda_K does through the soft output and through the last sweep nearly
// cancel, and an FP32 rounding of a constant would be common to all terms.
template <int HALF>
__device__ __forceinline__ void gram_axis_seed(const Params &P, const GramUser &user, double t, long o,
                                               double &sum_l, double &sum_d)
{
    constexpr int M = 1 << HALF;
    const float tf = (float)t;
    sum_l = sum_d = 0.0;
#pragma unroll
    for (int b = 0; b < HALF; ++b) {
        float d0 = INFINITY, d1 = INFINITY, l0 = 0.f, l1 = 0.f;
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const float l = (float)(2 * m - M + 1), d = (tf - l) * (tf - l);
            if (((m ^ (m >> 1)) >> (HALF - 1 - b)) & 1) {
                if (d < d1) { d1 = d; l1 = l; }
            } else {
                if (d < d0) { d0 = d; l0 = l; }
            }
        }
        const double dl = 2.0 * (double)(l1 - l0), D = fma(t, dl, (double)(l0 * l0 - l1 * l1));
        const float g = P.dllr ? global_ptr(P.dllr)[o + b]
                               : bce_grad((float)(user.c * D), global_ptr(P.bits)[o + b], P.inv_nbits);
        sum_l = fma((double)g, dl, sum_l);
        sum_d = fma((double)g, D, sum_d);
    }
}

__device__ __forceinline__ float2 gram_seed(const Params &P, float2 z, const GramUser &user, float d,
                                            float p, float lamK, long o, double &lamK_bar)
{
    if (!(user.c > 0.f)) return make_float2(0.f, 0.f);   // a zero column
    const double tr = user.a * z.x, ti = user.a * z.y;
    double lr, li, dr, di;   // sums over the bits of Re and Im
    if (P.Q == 2) {
        gram_axis_seed<1>(P, user, tr, o, lr, dr);
        gram_axis_seed<1>(P, user, ti, o + 1, li, di);
    } else if (P.Q == 4) {
        gram_axis_seed<2>(P, user, tr, o, lr, dr);
        gram_axis_seed<2>(P, user, ti, o + 2, li, di);
    } else {
        gram_axis_seed<3>(P, user, tr, o, lr, dr);
        gram_axis_seed<3>(P, user, ti, o + 3, li, di);
    }
    if (lamK > 0.f) {   // through rho = g / lambda and mu = p (t goes with 1 / mu)
        const double g = user.g, il = 1.0 / (double)lamK;
        lamK_bar = fma(P.llr_c * (dr + di), -g * il * il, lamK_bar);
        lamK_bar = fma(-(double)user.c * (tr * lr + ti * li), -g * d * ((double)d / p), lamK_bar);
    }
    const double s = user.c * user.a;
    return make_float2((float)(s * lr), (float)(s * li));
}

template <int UP, GramSymbols SY, int NW>
constexpr int grad_lanes()
{
    return SY == SY_NONE ? (UP == 32 ? 16 : 4) : gram_lanes<UP, SY, NW>();
}

// Adds the wave's sum of x to its partial sum of entry e.
__device__ __forceinline__ void add_part(double *part, int e, float x)
{
    const float t = wave_sum(x);
    if ((threadIdx.x & 63) == 0) part[e * GRAM_WAVES + (threadIdx.x >> 6)] += (double)t;
}

// The forward sweeps of a tile's vectors after gram_front: z after every sweep into zh
// (FP32) and, in FP64, the last one in the place of the matched filters.
template <int UP, GramSymbols SY, bool BOX, int NW>
__device__ __forceinline__ void grad_forward(const Params &P, long w0, int ns, int tsyms,
                                             double *lds, const GramUser *us, float2 *zh)
{
    constexpr int L = grad_lanes<UP, SY, NW>(), R = UP / L;
    using M = GramLds<UP, SY, NW>;
    const int U = P.U, K = P.K;
    const GramVector<L, NW> x(P, w0, ns);
    if (x.wave_idle) return;
    double *m = lds + x.sub * M::SUMS;
    const double2 *G = reinterpret_cast<const double2 *>(m + M::G);
    double2 *Q = reinterpret_cast<double2 *>(m + M::Q) + x.s * UP + x.i * R;
    float2 *zrow = zh + (size_t)(x.sub * tsyms + x.s) * K * U + x.i * R;
    double2 q[R], z[R];
#pragma unroll
    for (int r = 0; r < R; ++r) q[r] = Q[r];
    gram_run<UP, BOX, L>(P, x.w, x.i, G, us + x.sub * UP, q, z, [&](int k) {
        if (x.active) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (x.i * R + r < U) zrow[k * U + r] = make_float2((float)z[r].x, (float)z[r].y);
        }
    });
    if (x.active) {
#pragma unroll
        for (int r = 0; r < R; ++r) Q[r] = z[r];
    }
}

// The soft output of a tile and its adjoint, one (vector, user) per thread: z, the LLRs and
// the loss (training step), and dLoss/dz into A.
template <int UP, GramSymbols SY, bool TRAIN, int NW>
__device__ __forceinline__ void grad_seeds(const Params &P, long w0, int s0, int ns, int tsyms,
                                           const double *lds, const GramUser *us, float2 *A,
                                           double *part)
{
    using M = GramLds<UP, SY, NW>;
    const int U = P.U, K = P.K;
    const float lamK = P.lambda ? global_ptr(P.lambda)[K - 1] : P.lam_default;
    const int items = M::SG * ns * UP;
    float loss = 0.f;
    double lamK_bar = 0.0;
    for (int idx = threadIdx.x; idx < items; idx += GRAM_THREADS) {
        const int u = idx % UP, vec = idx / UP, sub = vec / ns, s = vec - sub * ns;
        const long w = w0 + sub, v = w * P.S + s0 + s, o = (v * U + u) * P.Q;
        float2 seed = make_float2(0.f, 0.f);
        if (u < U && w < P.W) {
            const GramUser user = us[sub * UP + u];
            float2 z;
            if constexpr (TRAIN) {
                const double2 z2 =
                    reinterpret_cast<const double2 *>(lds + sub * M::SUMS + M::Q)[s * UP + u];
                z = make_float2((float)z2.x, (float)z2.y);
                if (P.z) global_store2(P.z + v * U + u, z);
                float Lv[6];
                gram_llrs(P, z2, user, Lv);
#pragma unroll
                for (int b = 0; b < 6; ++b) {
                    if (b >= P.Q) break;
                    if (P.llr) global_ptr(P.llr)[o + b] = Lv[b];
                    loss += bce_term(Lv[b], global_ptr(P.bits)[o + b]);
                }
            } else {
                z = global_load2(P.zh_in + (v * K + K - 1) * U + u);
            }
            float p;
            const float d = gram_dinv(P, w, K - 1, u, user.g, lamK, &p);
            seed = gram_seed(P, z, user, d, p, lamK, o, lamK_bar);
        }
        A[(sub * tsyms + s) * UP + u] = seed;
    }
    add_part(part, K - 1, (float)lamK_bar);
    if constexpr (TRAIN) add_part(part, K + 1, loss);
}

// The reverse sweeps of a tile's vectors: L lanes each, lane i owning users i R ..; the
// seeds in A are replaced by the users' A_u.
template <int UP, GramSymbols SY, bool BOX, bool TRAIN, int NW>
__device__ __forceinline__ void grad_reverse(const Params &P, long w0, int s0, int ns, int tsyms,
                                             const double *lds, const GramUser *us, float2 *A,
                                             double *part, const float2 *zh)
{
    constexpr int L = grad_lanes<UP, SY, NW>(), R = UP / L;
    using M = GramLds<UP, SY, NW>;
    const int U = P.U, K = P.K;
    const GramVector<L, NW> x(P, w0, ns);
    if (x.wave_idle) return;
    const int i = x.i;
    const long w = x.w, v = w * P.S + s0 + x.s;
    const double2 *G =
        reinterpret_cast<const double2 *>(lds + x.sub * M::SUMS + M::G) + i * R;
    us += x.sub * UP;
    A += (x.sub * tsyms + x.s) * UP + i * R;
    // z after every sweep; users past U read a valid entry and are zeroed below
    const float2 *zrow = TRAIN ? zh + (size_t)(x.sub * tsyms + x.s) * K * U
                               : P.zh_in + (size_t)v * K * U;
    auto z_at = [&](int k, int r) {
        const float2 *p = zrow + k * U + min(i * R + r, U - 1);
        return TRAIN ? *p : global_load2(p);
    };
    double2 zb[R], wv[R], av[R];
    float2 znext[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const float2 sd = A[r];
        zb[r] = make_double2(sd.x, sd.y);
        wv[r] = av[r] = make_double2(0.0, 0.0);
        znext[r] = z_at(K - 1, r);
    }
    const float beta = P.beta;
    double beta_bar = 0.0;
    double d[R], lam = 0.0;
    if (!P.per_sweep) lam = gram_coefs<R>(P, w, 0, i, us, d);
    for (int k = K - 1; k >= 0; --k) {
        if (P.per_sweep) lam = gram_coefs<R>(P, w, k, i, us, d);
        // a user's update of this sweep: a = d (z_bar - w), 0 in a clipped component (whose
        // t = z_bar - w goes to beta_bar); z_bar then is w + p c_bar = z_bar - lambda a
        // (p = 1 - lambda d), or w = z_bar - t where clipped.  z_bar changes once per sweep,
        // so all but the FMA in w_u are formed before it and after it.  With d = 0 it is w
        // too: no user's a changes w_u then, as g_u + lambda is 0 with h_u = 0 or infinite
        // with lambda, for every user.
        float2 zn[R];
        double2 dm[R], sv[R], asum[R], tsum[BOX ? R : 1];
#pragma unroll
        for (int r = 0; r < R; ++r) {   // the row of the next sweep, ahead of its use
            zn[r] = i * R + r < U ? znext[r] : make_float2(0.f, 0.f);
            znext[r] = z_at(max(k - 1, 0), r);
            dm[r] = make_double2(d[r], d[r]);
            if constexpr (BOX) {
                if (!(fabsf(zn[r].x) < beta)) dm[r].x = 0.0;
                if (!(fabsf(zn[r].y) < beta)) dm[r].y = 0.0;
                tsum[r] = make_double2(0.0, 0.0);
            }
            sv[r] = make_double2(dm[r].x * zb[r].x, dm[r].y * zb[r].y);
            asum[r] = make_double2(0.0, 0.0);
        }
        static_for<UP / 4>([&](auto cc) {
            constexpr int c = UP / 4 - 1 - decltype(cc)::value;
            if (4 * c < U) {
                static_for<4>([&](auto uc) {
                    constexpr int u = 4 * c + 3 - decltype(uc)::value, o = u / R, n = u % R;
                    const double ar = fma(-dm[n].x, wv[n].x, sv[n].x);
                    const double ai = fma(-dm[n].y, wv[n].y, sv[n].y);
                    const double dr = group_bcast<L, o>(ar), di = group_bcast<L, o>(ai);
                    const double own = i == o ? 1.0 : 0.0;
                    asum[n].x = fma(own, ar, asum[n].x);
                    asum[n].y = fma(own, ai, asum[n].y);
                    if constexpr (BOX) {
                        tsum[n].x = fma(own, zb[n].x - wv[n].x, tsum[n].x);
                        tsum[n].y = fma(own, zb[n].y - wv[n].y, tsum[n].y);
                    }
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const double2 a = G[u * UP + r];
                        wv[r].x = fma(a.x, dr, fma(-a.y, di, wv[r].x));
                        wv[r].y = fma(a.x, di, fma(a.y, dr, wv[r].y));
                    }
                });
            }
        });
        double lam_bar = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            lam_bar = fma(-(double)zn[r].x, asum[r].x, fma(-(double)zn[r].y, asum[r].y, lam_bar));
            av[r].x += asum[r].x;
            av[r].y += asum[r].y;
            double2 step = make_double2(lam * asum[r].x, lam * asum[r].y);
            if constexpr (BOX) {
                if (!(fabsf(zn[r].x) < beta)) { step.x = tsum[r].x; beta_bar += zn[r].x > 0.f ? tsum[r].x : -tsum[r].x; }
                if (!(fabsf(zn[r].y) < beta)) { step.y = tsum[r].y; beta_bar += zn[r].y > 0.f ? tsum[r].y : -tsum[r].y; }
            }
            zb[r].x -= step.x;
            zb[r].y -= step.y;
            if (!(d[r] > 0.0)) zb[r] = wv[r];
        }
        add_part(part, k, x.active ? (float)lam_bar : 0.f);
    }
    if constexpr (BOX) add_part(part, K, x.active ? (float)beta_bar : 0.f);
    if (x.active) {
#pragma unroll
        for (int r = 0; r < R; ++r) A[r] = make_float2((float)av[r].x, (float)av[r].y);
    }
}

// dy = H A of a tile, two antennas a lane: the symbols of the tile dealt over the waves
// (NW = 4), or the wave's own subcarrier (NW = 1), four symbols at a time.
template <int UP, bool F16, int NW>
__device__ __forceinline__ void grad_dy(const Params &P, long w0, int s0, int ns, int tsyms,
                                        const float2 *A)
{
    const int U = P.U, B = P.B;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const long w = NW == 4 ? w0 : w0 + wave;
    if (w >= P.W) return;
    if (NW == 1) A += wave * tsyms * UP;
    const unsigned char *hb =
        static_cast<const unsigned char *>(P.H) + (size_t)w * U * B * cbytes<F16>();
    float2 *dy = P.dy + (w * P.S + s0) * B;
    constexpr int STEP = NW == 4 ? GRAM_WAVES : 1;
    for (int s = NW == 4 ? wave : 0; s < ns; s += 4 * STEP) {
        for (int b = 2 * lane; b < B; b += 128) {
            float4 acc[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int u0 = 0; u0 < U; u0 += 8) {   // eight users' entries in flight
                GramRaw<F16> raw[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    raw[j] = P.vec_ok ? gram_load<F16, true>(hb, min(u0 + j, U - 1), b, B)
                                      : gram_load<F16, false>(hb, min(u0 + j, U - 1), b, B);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (u0 + j >= U) break;
                    const float4 h = gram_pair<F16>(raw[j], false, b, B);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (s + q * STEP >= ns) break;
                        const float2 a = A[(s + q * STEP) * UP + u0 + j];
                        acc[q].x = fmaf(h.x, a.x, acc[q].x);
                        acc[q].y = fmaf(h.x, a.y, acc[q].y);
                        acc[q].z = fmaf(h.z, a.x, acc[q].z);
                        acc[q].w = fmaf(h.z, a.y, acc[q].w);
                        acc[q].x = fmaf(-h.y, a.y, acc[q].x);
                        acc[q].y = fmaf(h.y, a.x, acc[q].y);
                        acc[q].z = fmaf(-h.w, a.y, acc[q].z);
                        acc[q].w = fmaf(h.w, a.x, acc[q].w);
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (s + q * STEP >= ns) break;
                float2 *o = dy + (size_t)(s + q * STEP) * B + b;
                global_store2(o, make_float2(acc[q].x, acc[q].y));
                if (b + 1 < B) global_store2(o + 1, make_float2(acc[q].z, acc[q].w));
            }
        }
    }
}

template <int UP, GramSymbols SY, bool F16, int NW>
__device__ __forceinline__ void grad_front(const Params &P, long w0, int s0, int ns, double *lds,
                                           GramUser *us)
{
    const int sub = NW == 4 ? 0 : threadIdx.x >> 6;
    const long w = gram_subcarrier<NW>(P, w0);
    lds += sub * GramLds<UP, SY, NW>::SUMS;
    us += sub * UP;
    gram_dispatch<UP, F16>(P, [&](auto vec, auto half) {
        gram_front<UP, SY, F16, vec(), half(), NW>(P, w, s0, ns, lds, us);
    });
}

// LOOP: more tiles than workgroups.  Without the loop the values that it would keep across
// tiles free registers.
template <int UP, GramSymbols SY, bool F16, bool BOX, bool TRAIN, int NW, bool LOOP>
__global__ __launch_bounds__(GRAM_THREADS, 2) void k_gram_grad(Params P, int tsyms, int ntiles)
{
    extern __shared__ __align__(16) unsigned char smem[];
    using M = GradLds<UP, SY, TRAIN, NW>;
    const int K = P.K, E = K + (TRAIN ? 2 : 1);
    double *lds = reinterpret_cast<double *>(smem);
    GramUser *us = reinterpret_cast<GramUser *>(smem + M::US);
    float2 *A = reinterpret_cast<float2 *>(smem + M::A);
    double *part = reinterpret_cast<double *>(smem + M::part(tsyms));
    float2 *zh = reinterpret_cast<float2 *>(smem + M::zh(tsyms, K));
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int e = lane; e < K + 2; e += 64) part[e * GRAM_WAVES + wave] = 0.0;
    stagger_loads(P);
    const int per = (P.S + tsyms - 1) / tsyms;   // tiles per group of subcarriers
    auto tile = [&](int t) {
        const int g = per == 1 ? t : t / per, s0 = (t - g * per) * tsyms;
        const int ns = min(tsyms, P.S - s0);
        const long w0 = (long)g * M::SG;
        grad_front<UP, SY, F16, NW>(P, w0, s0, ns, lds, us);
        if constexpr (TRAIN) {
            grad_forward<UP, SY, BOX, NW>(P, w0, ns, tsyms, lds, us, zh);
            __syncthreads();
        }
        grad_seeds<UP, SY, TRAIN, NW>(P, w0, s0, ns, tsyms, lds, us, A, part);
        __syncthreads();
        grad_reverse<UP, SY, BOX, TRAIN, NW>(P, w0, s0, ns, tsyms, lds, us, A, part, zh);
        __syncthreads();
        if (P.dy) grad_dy<UP, F16, NW>(P, w0, s0, ns, tsyms, A);
    };
    if constexpr (LOOP) {
        for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
            tile(t);
            __syncthreads();   // the next tile reuses the LDS
        }
    } else {
        tile(blockIdx.x);
    }
    __syncthreads();
    float *out = P.partials + (size_t)blockIdx.x * E;
    for (int e = threadIdx.x; e < E; e += GRAM_THREADS) {
        double sum = 0.0;
        for (int q = 0; q < GRAM_WAVES; ++q) sum += part[e * GRAM_WAVES + q];
        store_partial(out + e, (float)sum);
    }
    finish_partials(P, E);
}

// Symbols per tile: all of them up to 16 (8 for the two-in-one tiles) while z after every
// sweep fits beside the rest, 64 KB for the workgroup (two or more a CU) where that leaves
// any, the device's limit where it does not.
template <int UP, GramSymbols SY, bool TRAIN, int NW>
static int grad_tile_symbols(const Params &p, size_t limit)
{
    using M = GradLds<UP, SY, TRAIN, NW>;
    int t = p.S <= 8 ? 8 : 16;
    while (t > 1 && t / 2 >= p.S) t /= 2;
    while (t > 1 && M::bytes(t, p.K, p.U) > (size_t)65536) t /= 2;
    return M::bytes(t, p.K, p.U) <= limit ? t : 0;
}

// max_blocks: the most workgroups whose partial sums fit the caller's scratch.
template <int UP, GramSymbols SY, bool F16, bool BOX, bool TRAIN, int NW>
static hipError_t launch_grad_k(const Params &p, int max_blocks, size_t limit, hipStream_t s)
{
    using M = GradLds<UP, SY, TRAIN, NW>;
    const int tsyms = grad_tile_symbols<UP, SY, TRAIN, NW>(p, limit);
    if (!tsyms) return hipErrorInvalidValue;
    const int ntiles = (p.W + M::SG - 1) / M::SG * ((p.S + tsyms - 1) / tsyms);
    const int most = (int)groups_per_launch(1, GRAM_THREADS);
    const int limited = max_blocks < most ? max_blocks : most;
    const int grid = ntiles < limited ? ntiles : limited;
    auto fn = grid < ntiles ? k_gram_grad<UP, SY, F16, BOX, TRAIN, NW, true>
                            : k_gram_grad<UP, SY, F16, BOX, TRAIN, NW, false>;
    const size_t lds = M::bytes(tsyms, p.K, p.U);
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    Params q = p;
    if (q.stagger > 0) {
        int per_cu = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per_cu, reinterpret_cast<const void *>(fn), GRAM_THREADS, lds);
        if (e != hipSuccess) return e;
        q.stagger_cap = per_cu * device_cu_count();
    }
    hipLaunchKernelGGL(fn, dim3(grid), dim3(GRAM_THREADS), lds, s, q, tsyms, ntiles);
    return hipGetLastError();
}

// A subcarrier per wave where there are enough of them and z after every sweep of a whole
// tile fits (see gram_waves), else four waves on one.
template <int UP, GramSymbols SY, bool F16, bool BOX, bool TRAIN>
static hipError_t launch_grad_w(const Params &p, int max_blocks, size_t limit, hipStream_t s)
{
    if constexpr (UP <= 16) {
        const int t = grad_tile_symbols<UP, SY, TRAIN, 1>(p, limit);
        if (grad_one_wave<TRAIN>(p) && t >= (p.S < 16 ? p.S : 16))
            return launch_grad_k<UP, SY, F16, BOX, TRAIN, 1>(p, max_blocks, limit, s);
    }
    return launch_grad_k<UP, SY, F16, BOX, TRAIN, 4>(p, max_blocks, limit, s);
}

template <int UP, bool TRAIN>
static hipError_t launch_grad_u(bool f16, const Params &p, int max_blocks, size_t limit,
                                hipStream_t s)
{
    constexpr GramSymbols S16 = TRAIN ? SY_16 : SY_NONE, S8 = TRAIN ? SY_8 : SY_NONE;
    if (p.S <= 8) {
        if (f16) return p.box ? launch_grad_w<UP, S8, true, true, TRAIN>(p, max_blocks, limit, s)
                              : launch_grad_w<UP, S8, true, false, TRAIN>(p, max_blocks, limit, s);
        return p.box ? launch_grad_w<UP, S8, false, true, TRAIN>(p, max_blocks, limit, s)
                     : launch_grad_w<UP, S8, false, false, TRAIN>(p, max_blocks, limit, s);
    }
    if (f16) return p.box ? launch_grad_w<UP, S16, true, true, TRAIN>(p, max_blocks, limit, s)
                          : launch_grad_w<UP, S16, true, false, TRAIN>(p, max_blocks, limit, s);
    return p.box ? launch_grad_w<UP, S16, false, true, TRAIN>(p, max_blocks, limit, s)
                 : launch_grad_w<UP, S16, false, false, TRAIN>(p, max_blocks, limit, s);
}

template <bool TRAIN>
static hipError_t launch_grad(bool f16, const Params &p, int max_blocks, size_t limit, hipStream_t s)
{
    if (p.U <= 8) return launch_grad_u<8, TRAIN>(f16, p, max_blocks, limit, s);
    if (p.U <= 16) return launch_grad_u<16, TRAIN>(f16, p, max_blocks, limit, s);
    return launch_grad_u<32, TRAIN>(f16, p, max_blocks, limit, s);
}

}  // namespace ocd
