// ocd_forms.h -- which shapes run in which form, and in how many launches (host only, no HIP).
#pragma once

namespace ocd {

// A launch takes fewer than 2^32 work-items: the most groups of `blocks` workgroups of
// `threads` threads that fit one (a grid with more goes out in several launches).
inline long groups_per_launch(long blocks, int threads)
{
    return 0xFFFFFFFFL / threads / blocks;
}

// Whether a detection carries the inner products h_u^H r through the Gram matrix
// (ocd_gram.h) instead of the residual.  Few users' channel fits the registers
// (ocd_forward_reg.hip), where the residual form takes 0.24-0.9 of the Gram form's time up
// to S = 2.  Elsewhere the contraction costs the same whatever K is, for 8, 16 or 32 users,
// and once for every 16 symbols, and the residual form grows with U K, from 17 users on
// (whose tiles of 32 x 32 hide less) with B U K.  Up to two tiles a compute unit the latency
// of a workgroup counts, which the Gram form's fewer steps shorten: 0.3-0.9 of the time on
// either side of the later lines.  Time of the Gram form over the residual form's where the
// lines keep the residual, FP32 (the first with the quicker FP32 products):
//   few updates          U = 4, K = 1, 2: 0.9-1.35; U = 9, K = 1, 2: 0.9-1.16; 40 x 17, K = 1 to
//                        4: 0.9-1.54; 64 x 24, K = 1, 2: 0.9-1.19
//   a tile a third full  128 x 4, K = 4, S = 3: 1.12, 256 x 4: 1.29; S = 7: 0.80, 0.86;
//                        512 x 20, K = 1: 1.07-1.74; from 3072 tiles on 64 x 9, K = 4: 1.03-
//                        1.14, 18 x 9 1.03-1.37, 26 x 9, K = 3: 1.25 (0.87-0.98 at 2400)
//   S = 17               128 x 12, K = 2: 1.19, K = 4: 0.84; 256 x 32, K = 2: 1.18, K = 4: 0.69;
//                        128 x 24, K = 2, 4: 1.65, 1.13; S = 14: 1.12, 0.77
inline bool gram_form(int B, int U, int W, int S, int K)
{
    const int n = U * K;
    const bool base = U <= 8 ? n >= 16 : U <= 16 ? n >= 20 : (long)B * n >= 4096;
    if (!base || B < 2 * U || (U <= 8 && S < 3 && B <= 256)) return false;
    const long tiles = (long)W * ((S + 15) / 16);
    if (U <= 8) return !(U <= 4 && S <= 4 && n < 24 && tiles > (B >= 128 ? 2048 : 12000));
    if (U <= 10 && B * U < 1024 && n < 50 && tiles > 3072) return false;
    if (S > 16)
        return tiles <= 512 || B > 256 || (U <= 16 ? K >= 3 : (long)B * n >= 24576);
    if (U <= 16) return true;
    return !(S >= 3 && n < 32) && !(U <= 24 && K <= 2 && S > 8 && tiles > 512);
}

// The same for the gradients, and for a detection that writes the history that an adjoint
// reads (so that the training step is the two launches bit for bit).  Their contraction,
// forward and reverse sweeps take one wave's registers for longer, and fewer of them run at
// once: past two tiles a compute unit the Gram form needs more work in the updates that it
// shortens.  Time of training step, adjoint over the residual form's on either side, at the
// worst of 520 to 2048 subcarriers:
//   U <= 8, S > 8    64 x 8, K = 2: 1.13, 1.11; K = 4: 0.91, 0.94; 32 x 8, K = 2: 1.30, 1.24
//   U <= 8, S = 17   64 x 8, K = 2: 1.18, 1.17; K = 4: 0.94, 1.02; 32 x 8, K = 4: 1.32, 1.28
//   U > 8, S > 8     100 x 12, K = 4: 1.18, 0.95; 128 x 16, K = 4: 0.94, 0.85; 128 x 32,
//                    K = 1: 1.0, 1.34; K = 2: 0.97, 0.85
//   U > 8, S = 17    128 x 16, K = 4: 1.54, 1.08; 256 x 16, K = 4: 1.10, 1.02; 128 x 32,
//                    K = 2: 1.63, 1.47; K = 4: 1.01, 1.17
//   S = 8            128 x 4, K = 4: 1.13, 1.25; 128 x 32, K = 1: 1.19, 1.25; 256 x 16, K = 2:
//                    1.11, 1.25
// Past 2048 subcarriers, one layer of the one-wave workgroups, few antennas or a tile that
// the users do not fill leave the residual form the faster; training step and adjoint at 2500
// to 14000 subcarriers, S = 4, K = 4:
//   residual         32 x 8 1.00-1.42, 1.12-1.62; 64 x 4 1.00-1.61, 1.13-1.82; 64 x 9
//                    0.84-1.39, 1.20-1.98; 32 x 16 0.76-1.29, 1.09-1.61
//   Gram             64 x 8 0.68-0.75, 0.77-1.25; 128 x 8 0.63-0.71, below 1; 64 x 16 0.63,
//                    up to 1.11; 64 x 24 0.57-0.73, 1.11-1.46
// (where one gains more than the other loses, the gradients stay in the Gram form).  Where
// workgroups take several tiles each, their loop costs registers, K = 4: 128 x 8 0.84, 1.46;
// 64 x 8 1.15, 2.05; 64 x 24 0.95, 1.78; against 64 x 16 0.57, 1.00; 128 x 24 0.95, 0.84; and
// 64 x 8, K = 20, 0.71, 1.17.
inline bool gram_gradient(int B, int U, int W, int S, int K)
{
    const int n = U * K;
    const long tiles = (long)W * ((S + 15) / 16), work = (long)B * n;
    if (!gram_form(B, U, 1, S, K)) return false;
    if (U <= 8 && S > 16) return tiles <= 256 || (n >= 24 && work >= 2048);
    if (tiles <= 512) return true;
    // more workgroups (of four subcarriers, or one) than the static scratch has partial sums for
    const long groups = U <= 16 ? tiles / 4 : tiles;
    if (groups > 262080 / (K + 1) && K <= 8 && (U <= 8 || (U > 16 && B * U < 2048))) return false;
    if (tiles > 2304 && U <= 16) {
        const int full = U <= 4 ? 1024 : U <= 8 ? 512 : U <= 12 ? 1024 : 520;
        if (B * U < full) return false;
    }
    if (U > 8 && U <= 16 && B > 128 && K <= 2 && S > 4) return false;
    if (S <= 8) return S <= 4 || !(U <= 4 ? n < 24 : U > 16 && K == 1);
    if (U <= 8) return n >= 24;
    return work >= (S <= 16 ? 8192 : 16384);
}

}  // namespace ocd
