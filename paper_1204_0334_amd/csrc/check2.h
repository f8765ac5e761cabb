// Check-node update (Algorithm 1, Eq. 3) with messages in base-2 units, for
// the decoders whose time goes into this arithmetic rather than into memory
// traffic: the on-chip block decoders (onchip.hip, onchip_wide.hip) and the
// convolutional-code decoders (sweep.hip, decode.hip).  A message x here is
// the LLR times log2(e), so the probability ratio of its two values is 2^x
// and the output magnitude the log2 of a ratio: the hardware's 2^x and log2
// apply without a scaling multiply on either side.  The decoders scale the
// channel LLRs once when they read them and the posteriors back when they
// write them; the clip at 30 becomes a clip at 30 log2(e).
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

#include "device.h"

namespace ldpc {

constexpr float kClip2 = 43.2808512266689f;   // 30 * log2(e)
constexpr float kLog2eF = 1.4426950408889634f;
constexpr float kLn2F = 0.6931471805599453f;

__device__ __forceinline__ float clip2(float x) { return __builtin_amdgcn_fmed3f(x, -kClip2, kClip2); }

// Posterior in natural units from the base-2 sum L = mu log2(e) + sum alpha: one
// rounding (with mu's part taken out first, and added back unscaled, there are
// two: up to 1.05 times the error against 64 bits once posteriors are large).
__device__ __forceinline__ float unscale2(float L) { return clip30(L * kLn2F); }

// Posterior in natural units from the base-2 sum S of the alphas alone and the
// channel LLR mu.  Where S can be had this is the better form: L's rounding,
// that of the sum with mu, does not come in.
__device__ __forceinline__ float posterior2(float S, float mu) { return fmaf(S, kLn2F, mu); }

// Eq. 3 for one row in base-2 units, in place: x[k] = beta of slot k on
// entry, alpha of slot k on return (k < d; the other slots are left with
// values nobody reads).  In terms of e = 2^-|beta|, the ratio of the two
// values' probabilities, inputs combine as (1, e) pairs: for the parity of
// two groups of bits with (even, odd) weights (A, W) and (B, V) these are
// (A B + W V, A V + W B), and |alpha| = log2(even / odd) over the other
// slots.  Every term is positive, so nothing cancels, a step of a sweep is
// two fused multiply-adds, and no input needs a reciprocal (A grows to 2^24
// at most, W stays above 2^-44).  The error of alpha against 64 bits, over
// rows of weight 6 to 24 and mean LLRs of 0.5 to 15, is 0.4-1.0 of that of
// the package decoder's (tanh, 1 - tanh) pairs.  Between the two steps a slot
// holds e (an unused slot 0, whose pair is the identity; it enters with x =
// 0, a positive sign).
// The slots are swept in NB blocks, so that only one block's suffix pairs are
// held at a time, at the cost of the products over the blocks behind.
template <int DC, int NB>
__device__ __forceinline__ void check2e_row(float (&x)[DC], int d) {
    constexpr int B = DC / NB;
    static_assert(B * NB == DC && B >= 2, "blocks of equal size");
    // the signs, slot k's in bit DC - 1 - k; then those of the outputs
    uint32_t sgn = 0;
#pragma unroll
    for (int k = 0; k < DC; ++k) {
        sgn = __builtin_amdgcn_alignbit(sgn, __float_as_uint(x[k]), 31);
        x[k] = k < d ? __builtin_amdgcn_exp2f(-fabsf(x[k])) : 0.0f;
    }
    sgn ^= (uint32_t)-(int32_t)(__builtin_popcount(sgn) & 1);
    // (A, W) of the slots behind each block
    float TA[NB], TW[NB];
    TA[NB - 1] = 1.0f;
    TW[NB - 1] = 0.0f;
#pragma unroll
    for (int b = NB - 2; b >= 0; --b) {
        float P = TA[b + 1], W = TW[b + 1];
#pragma unroll
        for (int i = B - 1; i >= 0; --i) {
            const float e = x[(b + 1) * B + i];
            if (b == NB - 2 && i == B - 1) {
                W = e;
            } else {
                const float t = fmaf(W, e, P);
                W = fmaf(P, e, W);
                P = t;
            }
        }
        TA[b] = P;
        TW[b] = W;
    }
    float PA = 1.0f, PW = 0.0f;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        // opaque, or the compiler would hold the pairs formed on the way to
        // (TA, TW) instead of forming them again
        if (b > 0) {
#pragma unroll
            for (int i = 0; i < B; ++i) asm volatile("" : "+v"(x[b * B + i]));
        }
        // suffix pairs of the block's slots (the last slot of all: the identity)
        float sA[B], sW[B];
        sA[B - 1] = TA[b];
        sW[B - 1] = TW[b];
#pragma unroll
        for (int i = B - 2; i >= 0; --i) {
            const float e = x[b * B + i + 1];
            if (b == NB - 1 && i == B - 2) {
                sA[i] = 1.0f;
                sW[i] = e;
            } else {
                sA[i] = fmaf(sW[i + 1], e, sA[i + 1]);
                sW[i] = fmaf(sA[i + 1], e, sW[i + 1]);
            }
        }
        float rA = 0.0f, rW = 0.0f;
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const int k = b * B + i;
            float eA, eW;
            if (k == 0) {
                eA = sA[0];
                eW = sW[0];
            } else if (k == DC - 1) {
                eA = PA;
                eW = PW;
            } else if (k == 1) {
                eA = fmaf(PW, sW[i], sA[i]);
                eW = fmaf(PW, sA[i], sW[i]);
            } else {
                eA = fmaf(PA, sA[i], PW * sW[i]);
                eW = fmaf(PA, sW[i], PW * sA[i]);
            }
            const float e = x[k];
            if (k == 0) {
                PW = e;
            } else if (k < DC - 1) {
                const float t = fmaf(PW, e, PA);
                PW = fmaf(PA, e, PW);
                PA = t;
            }
            // the ratio of slot k - 1 here and the logarithms after the loop: the
            // transcendental unit's results are not waited for one by one
            if (i > 0) x[k - 1] = rA * rW;
            rA = eA;
            rW = __builtin_amdgcn_rcpf(eW);
        }
        x[b * B + B - 1] = rA * rW;
#pragma unroll
        for (int i = 0; i < B; ++i) x[b * B + i] = __builtin_amdgcn_logf(x[b * B + i]);
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const int k = b * B + i;
            x[k] = __builtin_copysignf(x[k], __uint_as_float(sgn << (31 - (DC - 1 - k))));
        }
    }
}

// Learned min-sum rule (the package decoder's RULE 1) in base-2 units:
// alpha_k = w_k s_k max(m_k - b_k, 0), m_k the smallest |beta| of the row's
// other edges (|beta| <= 30 log2 e already), s_k the product of their signs
// (no beta is -0, so the sign bit is beta < 0); w[2k], w[2k+1] = (scale,
// offset) of slot k's block, the offset in natural units (scaled here).  The
// second minimum is the median of a value and the two minima so far, and an
// edge that holds the minimum is one whose magnitude equals it (with a tie
// the two minima are equal), so no index is kept.  out may be in.  BASE2 =
// false: all in natural units, and -0 among the betas, as the package decoder.
template <int DC, bool BASE2 = true>
__device__ __forceinline__ void nms2_row(const float (&in)[DC], int d, const float* __restrict__ w,
                                         float (&out)[DC]) {
    float min1 = __builtin_inff(), min2 = __builtin_inff();
    uint32_t sgn = 0;   // slot k's sign in bit DC - 1 - k
#pragma unroll
    for (int k = 0; k < DC; ++k) {
        if (k < d) {
            const float m = fabsf(in[k]);
            min2 = __builtin_amdgcn_fmed3f(m, min1, min2);
            min1 = fminf(m, min1);
            sgn = __builtin_amdgcn_alignbit(sgn, __float_as_uint(BASE2 ? in[k] : in[k] + 0.0f), 31);
        } else {
            sgn <<= 1;
        }
    }
    sgn ^= (uint32_t)-(int32_t)(__builtin_popcount(sgn) & 1);
#pragma unroll
    for (int k = 0; k < DC; ++k) {
        if (k < d) {
            const float m = fabsf(in[k]) == min1 ? min2 : min1;
            const float v = fmaxf(m - (BASE2 ? w[2 * k + 1] * kLog2eF : w[2 * k + 1]), 0.0f);
            // rounded before it is added to a sum: the sums are the same whether a
            // message comes from a register or from another compute unit
            {
#pragma clang fp contract(off)
                out[k] = w[2 * k] * __builtin_copysignf(v, __uint_as_float(sgn << (32 - DC + k)));
            }
        }
    }
}

}  // namespace ldpc
