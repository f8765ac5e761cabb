// Training step of the learned min-sum decoder with a frame on one compute
// unit (gfx950), for full bases of 3 rows, and of 4 rows of weight 24.
//
// The message-package form (decode.hip) passes every message through memory
// eight times an iteration: forward, each iteration's alphas and betas are
// written and read; backward they are read again beside their gradients.
// Here one workgroup takes one frame through all iterations.  Thread i owns
// check rows (j, i + q*TB) and keeps their edges' messages in registers; two
// arrays of n floats in LDS carry messages from rows to rows.
//
// What the backward pass needs of a check row is not its betas but which
// edges hold the two smallest magnitudes, those magnitudes, and the signs
// (the minimum's gradient reaches no other edge): three words per row and
// iteration (four with rows of weight 24) instead of two floats per edge.  With the posteriors, from which
// the backward pass forms dloss/dL, that is 60 bytes per iteration and place
// of a base column of a 3 x 6 code, written once and read once.
//
// Forward, bit for bit as the package form: alpha by the learned rule (natural
// units), beta_k = clip(mu + (pre + suf)) with the other two edges' alphas
// added in order of the base rows, L = mu + ((a0 + a1) + a2).  Rows of base
// rows 1 and 2 publish their alphas, read each other's, base row 0's threads
// form L and their betas and publish a0 and mu in place, and base rows 1 and 2
// form theirs: four barriers per iteration (4 rows: train_forward4_kernel).
//
// Backward: LDS holds, per variable, D = dloss/dL + the sum of the gradients
// that reached its edges' betas; an edge's dalpha is D less its own.  An
// iteration reads D from one array and forms the next one's in the other
// (dloss/dL first, then base row by base row the two edges per row that a
// gradient reaches).  The weight gradients are summed per wavefront in
// registers, over many wavefronts in LDS, and written once per base row and
// iteration.  What memory holds
// is loaded a step ahead (without that the backward pass took a fifth longer).
//
// 3 x 6, p = 3060, 1024 frames, 12 iterations: forward 0.72 ms, backward
// 0.90 ms as traced, the sums over frames below 0.01 ms; loss and gradients
// together 1.62 ms untraced, 5.50 ms in the package form.  2.3 GB
// pass each way, 0.45 ms at the rate of a large copy; the rest is the
// workgroup's own arithmetic and LDS traffic between barriers, which one
// workgroup per compute unit (147 KB of LDS) does not hide.
#include <hip/hip_runtime.h>

#include "check2.h"
#include "device.h"
#include "internal.h"
#include "train.h"

namespace ldpc {

constexpr int kTrRows = 4, kTrSlots = 24, kTrWaves = 16;

// words kept per row: the minima, their edges and the signs (rows of weight
// above 18: the signs in a word of their own)
constexpr int tr_words(int dc) { return dc <= 18 ? 3 : 4; }

struct TrainArgs {
    const float* llr;      // [gamma][n] (forward)
    const float* w;        // [T][blocks][2]
    const float* dloss;    // [T] (backward)
    float* rows;           // [gamma][T][words][rows][p]: minimum, second minimum, edges and signs
    float* post;           // [gamma][T][n]: posteriors, by place
    float* lpart;          // [T][gamma]: loss sums
    float* gpart;          // [T][gamma][parts][blocks][2]
    float inv_count;
    int32_t n, p, T, gamma;
    int32_t parts;         // partial sums of a frame: one, or one per wavefront
    // Columns are kept rotated by base row 0's shifts (place l p + u holds
    // variable l p + (u + a_0l) mod p), so a row (0, s) meets the places l p +
    // s.  Edge slot k of base row j (index j * kTrSlots + k): 4 times its
    // shift less base row 0's; rot4[k]: 4 a_0k
    uint32_t sh4[kTrRows * kTrSlots], rot4[kTrSlots];
};

__device__ __forceinline__ float* tr_at(float* base, uint32_t byte) {
    return reinterpret_cast<float*>(reinterpret_cast<char*>(base) + byte);
}
__device__ __forceinline__ const float* tr_at(const float* base, uint32_t byte) {
    return reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + byte);
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// Sums of N values over a wavefront: v[i] returns the sum of value 4 i + (lane
// & 3), i < N / 4.  Two halving exchanges within groups of four lanes, then
// one sum per group position.
template <int N>
__device__ __forceinline__ void wave_sums(float (&v)[N]) {
    static_assert(N % 4 == 0, "groups of four");
    const bool odd = threadIdx.x & 1, high = threadIdx.x & 2;
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
        const float keep = odd ? v[2 * i + 1] : v[2 * i], send = odd ? v[2 * i] : v[2 * i + 1];
        v[i] = keep + dpp<0xB1>(send);   // from lane ^ 1
    }
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        const float keep = high ? v[2 * i + 1] : v[2 * i], send = high ? v[2 * i] : v[2 * i + 1];
        v[i] = keep + dpp<0x4E>(send);   // from lane ^ 2
    }
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        v[i] += dpp<0x124>(v[i]);        // rotated by 4, by 8 within 16 lanes
        v[i] += dpp<0x128>(v[i]);
        v[i] += __shfl_xor(v[i], 16);
        v[i] += __shfl_xor(v[i], 32);
    }
}

__device__ __forceinline__ float wave_sum_all(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// log(1 + exp(-L)); log(1 + x) as x log(u) / (u - 1), u = 1 + x rounded, which
// is accurate for small x too (Kahan)
__device__ __forceinline__ float softplus_neg_tr(float L) {
    const float x = __expf(-fabsf(L)), u = 1.0f + x;
    const float r = x * (kLn2F * __builtin_amdgcn_logf(u)) * __builtin_amdgcn_rcpf(u - 1.0f);
    return fmaxf(-L, 0.0f) + (u == 1.0f ? x : r);
}

// 1 / (1 + exp(L)), the reciprocal refined once
__device__ __forceinline__ float sigmoid_neg(float L) {
    const float d = fminf(1.0f + __expf(L), 1e37f);
    const float r = __builtin_amdgcn_rcpf(d);
    return fmaf(fmaf(-d, r, 1.0f), r, r);
}

// A check row's forward pass.  flip: bit DC - 1 - k, the sign of the product of
// the other edges of slot k; par: of all.
template <int DC>
struct TrRow {
    float m1, m2;
    uint32_t edges, flip, par;   // edges: i1, i2 << 5, unclipped << 10 and << 11

    // x: betas before the clip on entry, alphas on return
    __device__ __forceinline__ void update(float (&x)[DC], const float* __restrict__ w) {
        m1 = m2 = __builtin_inff();
        int i1 = 0, i2 = 0;
        uint32_t sgn = 0, cut = 0;   // slot k's sign, whether it is clipped: bit DC - 1 - k
#pragma unroll
        for (int k = 0; k < DC; ++k) {
            const float b = x[k] + 0.0f;   // no -0: the sign bit is beta < 0
            sgn = __builtin_amdgcn_alignbit(sgn, __float_as_uint(b), 31);
            cut = __builtin_amdgcn_alignbit(cut, __float_as_uint(kClip - fabsf(b)), 31);
            const float m = fminf(fabsf(b), kClip);
            const bool lt1 = m < m1, lt2 = m < m2;
            i2 = lt1 ? i1 : lt2 ? k : i2;
            i1 = lt1 ? k : i1;
            m2 = __builtin_amdgcn_fmed3f(m, m1, m2);
            m1 = fminf(m, m1);
        }
        par = (uint32_t)__builtin_popcount(sgn) & 1u;
        flip = (sgn ^ (0u - par)) & ((1u << DC) - 1u);
        edges = (uint32_t)i1 | (uint32_t)i2 << 5 | (~(cut >> (DC - 1 - i1)) & 1u) << 10 |
                (~(cut >> (DC - 1 - i2)) & 1u) << 11;
#pragma unroll
        for (int k = 0; k < DC; ++k) {
            const float v = fmaxf((k == i1 ? m2 : m1) - w[2 * k + 1], 0.0f);
            x[k] = w[2 * k] * __builtin_copysignf(v, __uint_as_float(flip << (32 - DC + k)));
        }
    }
    __device__ __forceinline__ void store(float* rows, int nj, int j, int p, uint32_t s4) const {
        *tr_at(rows + (size_t)j * p, s4) = m1;
        *tr_at(rows + (size_t)(nj + j) * p, s4) = m2;
        if constexpr (tr_words(DC) == 3) {
            *tr_at(rows + (size_t)(2 * nj + j) * p, s4) = __uint_as_float(edges | flip << 12 | par << 30);
        } else {
            *tr_at(rows + (size_t)(2 * nj + j) * p, s4) = __uint_as_float(edges);
            *tr_at(rows + (size_t)(3 * nj + j) * p, s4) = __uint_as_float(flip | par << 30);
        }
    }
};

template <int NQ, int DC>
__global__ void __launch_bounds__(1024) train_forward_kernel(const TrainArgs A) {
    extern __shared__ float lds[];   // X [n], Y [n], loss sums [waves]
    constexpr int kNJ = 3;
    const int n = A.n, p = A.p, tid = threadIdx.x, TB = blockDim.x;
    float* X = lds;
    float* Y = lds + n;
    float* part = lds + 2 * n;
    const uint32_t p4 = 4u * (uint32_t)p, TB4 = 4u * (uint32_t)TB;
    const size_t f = blockIdx.x;
    const float* __restrict__ mu = A.llr + f * n;

    // place of the variable that edge slot k of row (j, s) meets
    auto var4 = [&](uint32_t s4, int j, int k) -> uint32_t {
        if (j == 0) return (uint32_t)k * p4 + s4;
        const uint32_t t = s4 + A.sh4[j * kTrSlots + k];
        return (uint32_t)k * p4 + min(t, t - p4);
    };
    // channel LLR of the variable at place v4 of column k
    auto mu_at = [&](uint32_t v4, int k) -> float {
        const uint32_t t = v4 + A.rot4[k] - (uint32_t)k * p4;
        return *tr_at(mu, (uint32_t)k * p4 + min(t, t - p4));
    };
    float al[kNJ][NQ][DC];   // beta (before the clip) or alpha of the thread's edges
    float mu0[NQ][DC];           // channel LLRs of base row 0's edges
#pragma unroll
    for (int j = 0; j < kNJ; ++j)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const uint32_t s4 = 4u * (uint32_t)tid + (uint32_t)q * TB4;
#pragma unroll
            for (int k = 0; k < DC; ++k) al[j][q][k] = s4 < p4 ? mu_at(var4(s4, j, k), k) : 0.0f;
        }
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int k = 0; k < DC; ++k) mu0[q][k] = al[0][q][k];

    for (int t = 1; t <= A.T; ++t) {
        uint32_t tid4 = 4u * (uint32_t)tid;
        asm volatile("" : "+v"(tid4));   // the edges' variables are worked out again, not held
        float* rows = A.rows + (f * A.T + (t - 1)) * (3 * kNJ) * (size_t)p;
        // check rows
#pragma unroll
        for (int j = 0; j < kNJ; ++j) {
            const float* w = A.w + ((size_t)(t - 1) * kNJ + j) * DC * 2;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const uint32_t s4 = tid4 + (uint32_t)q * TB4;
                if (s4 < p4) {
                    TrRow<DC> row;
                    row.update(al[j][q], w);
                    row.store(rows, kNJ, j, p, s4);
                }
            }
        }
        // variables
        auto each = [&](int j, auto&& act) {
            if (DC > 9) asm volatile("" : "+v"(tid4));   // registers are scarce: nor held between the steps
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const uint32_t s4 = tid4 + (uint32_t)q * TB4;
                if (s4 < p4) {
#pragma unroll
                    for (int k = 0; k < DC; ++k) act(q, k, var4(s4, j, k));
                }
            }
        };
        each(1, [&](int q, int k, uint32_t v) { *tr_at(X, v) = al[1][q][k]; });
        each(2, [&](int q, int k, uint32_t v) { *tr_at(Y, v) = al[2][q][k]; });
        __syncthreads();
        each(1, [&](int q, int k, uint32_t v) { al[1][q][k] = *tr_at(Y, v); });   // a2
        each(2, [&](int q, int k, uint32_t v) { al[2][q][k] = *tr_at(X, v); });   // a1
        __syncthreads();
        float lsum = 0.0f;
        float* post = A.post + (f * A.T + (t - 1)) * (size_t)n;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const uint32_t s4 = tid4 + (uint32_t)q * TB4;
            if (s4 < p4) {
                constexpr int B = DC % 6 == 0 ? 6 : 3;   // slots whose reads go out together
#pragma unroll
                for (int k0 = 0; k0 < DC; k0 += B) {
                    uint32_t v[B];
                    float a1[B], a2[B];
#pragma unroll
                    for (int i = 0; i < B; ++i) {
                        v[i] = var4(s4, 0, k0 + i);
                        a1[i] = *tr_at(X, v[i]);
                        a2[i] = *tr_at(Y, v[i]);
                    }
#pragma unroll
                    for (int i = 0; i < B; ++i) {
                        const float a0 = al[0][q][k0 + i], m = mu0[q][k0 + i];
                        *tr_at(X, v[i]) = a0;
                        *tr_at(Y, v[i]) = m;
                        const float L = m + ((a0 + a1[i]) + a2[i]);
                        *tr_at(post, v[i]) = L;
                        lsum += softplus_neg_tr(L);
                        al[0][q][k0 + i] = m + (a2[i] + a1[i]);
                    }
                }
            }
        }
        lsum = wave_sum_all(lsum);
        if ((tid & 63) == 0) part[tid >> 6] = lsum;
        __syncthreads();
        if (t < A.T) {
            each(1, [&](int q, int k, uint32_t v) { al[1][q][k] = *tr_at(Y, v) + (*tr_at(X, v) + al[1][q][k]); });
            each(2, [&](int q, int k, uint32_t v) { al[2][q][k] = *tr_at(Y, v) + (*tr_at(X, v) + al[2][q][k]); });
        }
        if (tid == 0) {
            float sum = 0.0f;
            for (int i = 0; i < TB / 64; ++i) sum += part[i];
            A.lpart[(size_t)(t - 1) * A.gamma + f] = sum;
        }
        __syncthreads();
    }
}

// The same for bases of 4 rows.  One array carries the sums along the base
// rows, downwards the suffixes and upwards the prefixes that the package form
// adds (pre + suf), and the other holds the channel LLRs: seven steps per
// iteration, seven barriers, whose chain bounds it.  4 x 24, 18 iterations, 223
// frames, loss and gradients: p = 512 2580 us in the package form, 709 here; p
// = 653 (768 threads, 31 values spilled) 3229 and 1223.
template <int DC, int MAXT>
__global__ void __launch_bounds__(MAXT) train_forward4_kernel(const TrainArgs A) {
    extern __shared__ float lds[];   // X [n], channel LLRs by place [n], loss sums [waves]
    constexpr int kNJ = 4;
    const int n = A.n, p = A.p, tid = threadIdx.x, TB = blockDim.x;
    float* X = lds;
    float* M = lds + n;
    float* part = lds + 2 * n;
    const uint32_t p4 = 4u * (uint32_t)p;
    const size_t f = blockIdx.x;
    const float* __restrict__ mu = A.llr + f * n;
    const bool own = 4u * (uint32_t)tid < p4;
    auto var4 = [&](uint32_t s4, int j, int k) -> uint32_t {
        if (j == 0) return (uint32_t)k * p4 + s4;
        const uint32_t t = s4 + A.sh4[j * kTrSlots + k];
        return (uint32_t)k * p4 + min(t, t - p4);
    };
    float al[kNJ][DC], sf1[DC], sf2[DC];
    if (own) {
        const uint32_t s4 = 4u * (uint32_t)tid;
#pragma unroll
        for (int k = 0; k < DC; ++k) {
            const uint32_t t = s4 + A.rot4[k];
            al[0][k] = *tr_at(mu, (uint32_t)k * p4 + min(t, t - p4));
        }
#pragma unroll
        for (int k = 0; k < DC; ++k) *tr_at(M, (uint32_t)k * p4 + s4) = al[0][k];
    }
    __syncthreads();
#pragma unroll
    for (int j = 1; j < kNJ; ++j)
#pragma unroll
        for (int k = 0; k < DC; ++k) al[j][k] = own ? *tr_at(M, var4(4u * (uint32_t)tid, j, k)) : 0.0f;

    for (int t = 1; t <= A.T; ++t) {
        float* rows = A.rows + (f * A.T + (t - 1)) * (tr_words(DC) * kNJ) * (size_t)p;
        float* post = A.post + (f * A.T + (t - 1)) * (size_t)n;
        if (own) {
#pragma unroll
            for (int j = 0; j < kNJ; ++j) {
                TrRow<DC> row;
                row.update(al[j], A.w + ((size_t)(t - 1) * kNJ + j) * DC * 2);
                row.store(rows, kNJ, j, p, 4u * (uint32_t)tid);
            }
        }
        // each edge of base row j: its place, worked out again at every step
        auto each = [&](int j, auto&& act) {
            uint32_t s4 = 4u * (uint32_t)tid;
            asm volatile("" : "+v"(s4));
            if (own) {
                constexpr int B = 6;   // edges whose reads go out together
#pragma unroll
                for (int k0 = 0; k0 < DC; k0 += B) {
                    uint32_t v[B];
                    float x[B];
#pragma unroll
                    for (int i = 0; i < B; ++i) {
                        v[i] = var4(s4, j, k0 + i);
                        x[i] = *tr_at(X, v[i]);
                    }
#pragma unroll
                    for (int i = 0; i < B; ++i) act(k0 + i, v[i], x[i]);
                }
            }
        };
        if (own) {
#pragma unroll
            for (int k = 0; k < DC; ++k) *tr_at(X, var4(4u * (uint32_t)tid, 3, k)) = al[3][k];
        }
        __syncthreads();
        each(2, [&](int k, uint32_t v, float x) { sf2[k] = x; *tr_at(X, v) = x + al[2][k]; });
        __syncthreads();
        each(1, [&](int k, uint32_t v, float x) { sf1[k] = x; *tr_at(X, v) = x + al[1][k]; });
        __syncthreads();
        each(0, [&](int k, uint32_t v, float x) {
            *tr_at(X, v) = al[0][k];
            al[0][k] = *tr_at(M, v) + x;
        });
        __syncthreads();
        each(1, [&](int k, uint32_t v, float x) {
            *tr_at(X, v) = x + al[1][k];
            al[1][k] = *tr_at(M, v) + (x + sf1[k]);
        });
        __syncthreads();
        each(2, [&](int k, uint32_t v, float x) {
            *tr_at(X, v) = x + al[2][k];
            al[2][k] = *tr_at(M, v) + (x + sf2[k]);
        });
        __syncthreads();
        float lsum = 0.0f;
        each(3, [&](int k, uint32_t v, float x) {
            const float m = *tr_at(M, v), L = m + (x + al[3][k]);
            *tr_at(post, v) = L;
            lsum += softplus_neg_tr(L);
            al[3][k] = m + x;
        });
        lsum = wave_sum_all(lsum);
        if ((tid & 63) == 0) part[tid >> 6] = lsum;
        __syncthreads();
        if (tid == 0) {
            float sum = 0.0f;
            for (int i = 0; i < TB / 64; ++i) sum += part[i];
            A.lpart[(size_t)(t - 1) * A.gamma + f] = sum;
        }
    }
}

// ONE: the weight gradients of a frame in one sum (over its wavefronts, in LDS),
// else one per wavefront.
template <int kNJ, int NQ, int DC, int MAXT, bool ONE>
__global__ void __launch_bounds__(MAXT) train_backward_kernel(const TrainArgs A) {
    extern __shared__ float lds[];   // two arrays of n: D of this iteration, of the one before
    constexpr int NV = (2 * DC + 3) / 4 * 4;   // (dw, db) of a base row's slots, filled up to fours
    const int n = A.n, p = A.p, tid = threadIdx.x, TB = blockDim.x;
    const uint32_t p4 = 4u * (uint32_t)p, TB4 = 4u * (uint32_t)TB, n4 = 4u * (uint32_t)n;
    const size_t f = blockIdx.x;
    // place of the variable that edge slot k of row (j, s) meets; of a slot
    // that differs from lane to lane, the shifts from a copy in LDS
    auto var4 = [&](uint32_t s4, int j, int k) -> uint32_t {
        if (j == 0) return (uint32_t)k * p4 + s4;
        const uint32_t t = s4 + A.sh4[j * kTrSlots + k];
        return (uint32_t)k * p4 + min(t, t - p4);
    };
    uint32_t* shifts = reinterpret_cast<uint32_t*>(lds + 2 * n);
    float* red = lds + 2 * n + kTrRows * kTrSlots;
    int phase = 0;
    for (int i = tid; i < kNJ * DC; i += TB) shifts[i] = A.sh4[i / DC * kTrSlots + i % DC];
    auto var4_at = [&](uint32_t s4, int j, uint32_t k) -> uint32_t {
        if (j == 0) return k * p4 + s4;
        const uint32_t t = s4 + shifts[j * DC + k];
        return k * p4 + min(t, t - p4);
    };
    // gradients that reached the row's betas (two edges at most) and their slots
    float g1[kNJ][NQ], g2[kNJ][NQ];
    uint32_t at[kNJ][NQ];
#pragma unroll
    for (int j = 0; j < kNJ; ++j)
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            g1[j][q] = g2[j][q] = 0.0f;
            at[j][q] = 0u;
        }
    // what memory holds is read a step ahead: the posteriors of the iteration
    // before the next, the words of the next base row
    float L[NQ][DC], m1[NQ], m2[NQ];
    constexpr int kWords = tr_words(DC);
    uint32_t word[NQ], signs[NQ];
    auto load_posteriors = [&](int t, uint32_t tid4) {
        const float* post = A.post + (f * A.T + (t - 1)) * (size_t)n;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const uint32_t s4 = tid4 + (uint32_t)q * TB4;
#pragma unroll
            for (int k = 0; k < DC; ++k) L[q][k] = s4 < p4 ? *tr_at(post + (size_t)k * p, s4) : 0.0f;
        }
    };
    auto load_rows = [&](int t, int j, uint32_t tid4) {
        const float* rows = A.rows + (f * A.T + (t - 1)) * (kWords * kNJ) * (size_t)p;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const uint32_t s4 = tid4 + (uint32_t)q * TB4;
            m1[q] = m2[q] = 0.0f;
            word[q] = signs[q] = 0u;
            if (s4 < p4) {
                m1[q] = *tr_at(rows + (size_t)j * p, s4);
                m2[q] = *tr_at(rows + (size_t)(kNJ + j) * p, s4);
                word[q] = __float_as_uint(*tr_at(rows + (size_t)(2 * kNJ + j) * p, s4));
                if (kWords == 4) signs[q] = __float_as_uint(*tr_at(rows + (size_t)(3 * kNJ + j) * p, s4));
            }
        }
    };
    // dloss/dL of iteration t, from its posteriors, into the array at byte `to`
    auto start = [&](int t, uint32_t to, uint32_t tid4) {
        const float scale = A.dloss[t - 1] * A.inv_count;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const uint32_t s4 = tid4 + (uint32_t)q * TB4;
            if (s4 < p4) {
#pragma unroll
                for (int k = 0; k < DC; ++k)
                    *tr_at(lds, to + (uint32_t)k * p4 + s4) = -scale * sigmoid_neg(L[q][k]);
            }
        }
    };
    uint32_t cur = 0;
    load_posteriors(A.T, 4u * (uint32_t)tid);
    load_rows(A.T, 0, 4u * (uint32_t)tid);
    start(A.T, cur, 4u * (uint32_t)tid);
    if (A.T > 1) load_posteriors(A.T - 1, 4u * (uint32_t)tid);
    for (int t = A.T; t >= 1; --t) {
        uint32_t tid4 = 4u * (uint32_t)tid;
        asm volatile("" : "+v"(tid4));
        const uint32_t next = n4 - cur;
        if (t > 1) {
            start(t - 1, next, tid4);
            if (t > 2) load_posteriors(t - 2, tid4);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kNJ; ++j) {
            const float* w = A.w + ((size_t)(t - 1) * kNJ + j) * DC * 2;
            float c1[NQ], c2[NQ];
            uint32_t cw[NQ], cs[NQ];   // edges; flip in the low bits, par in bit 30 (18)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                c1[q] = m1[q];
                c2[q] = m2[q];
                cw[q] = word[q];
                cs[q] = kWords == 4 ? signs[q] : word[q] >> 12;
            }
            if (j + 1 < kNJ)
                load_rows(t, j + 1, tid4);
            else if (t > 1)
                load_rows(t - 1, 0, tid4);
            float sum[NV];
#pragma unroll
            for (int i = 0; i < NV; ++i) sum[i] = 0.0f;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const uint32_t s4 = tid4 + (uint32_t)q * TB4;
                if (s4 < p4) {
                    const uint32_t i1 = cw[q] & 31u, i2 = cw[q] >> 5 & 31u, flip = cs[q];
                    const uint32_t o1 = at[j][q] & 31u, o2 = at[j][q] >> 5 & 31u;
                    float D[DC];
#pragma unroll
                    for (int k = 0; k < DC; ++k) D[k] = *tr_at(lds, cur + var4(s4, j, k));
                    const uint32_t v1 = next + var4_at(s4, j, i1), v2 = next + var4_at(s4, j, i2);
                    float G1 = 0.0f, G2 = 0.0f;
#pragma unroll
                    for (int k = 0; k < DC; ++k) {
                        // dalpha with the sign of the other edges' product
                        float da = D[k] - ((uint32_t)k == o1 ? g1[j][q] : (uint32_t)k == o2 ? g2[j][q] : 0.0f);
                        da = __uint_as_float(__float_as_uint(da) ^ (flip << (32 - DC + k) & 0x80000000u));
                        const bool is1 = (uint32_t)k == i1;
                        const float a = (is1 ? c2[q] : c1[q]) - w[2 * k + 1];
                        const float gk = a >= 0.0f ? da * w[2 * k] : 0.0f;
                        sum[2 * k] = fmaf(da, fmaxf(a, 0.0f), sum[2 * k]);
                        sum[2 * k + 1] -= gk;
                        G1 += is1 ? 0.0f : gk;
                        G2 = is1 ? gk : G2;
                    }
                    // the minimum's gradient to the edge that holds it (the second
                    // minimum's for that edge's own output), unless clipped
                    const uint32_t par = cs[q] >> (kWords == 4 ? 30 : 18) & 1u;
                    const uint32_t n1 = (flip >> (DC - 1 - i1) & 1u) ^ par, n2 = (flip >> (DC - 1 - i2) & 1u) ^ par;
                    float r1 = (cw[q] >> 10 & 1u) && c1[q] != 0.0f ? G1 : 0.0f;
                    float r2 = (cw[q] >> 11 & 1u) && c2[q] != 0.0f ? G2 : 0.0f;
                    r1 = n1 ? -r1 : r1;
                    r2 = n2 ? -r2 : r2;
                    g1[j][q] = r1;
                    g2[j][q] = r2;
                    at[j][q] = cw[q];
                    if (t > 1) {
                        // base row j's only updates of these variables
                        const float x1 = *tr_at(lds, v1), x2 = *tr_at(lds, v2);
                        *tr_at(lds, v1) = x1 + r1;
                        *tr_at(lds, v2) = x2 + r2;
                    }
                }
            }
            wave_sums<NV>(sum);
            float* part = A.gpart + ((size_t)(t - 1) * A.gamma + f) * A.parts * (kNJ * DC * 2) + j * DC * 2;
            if constexpr (ONE) {
                // the wavefronts' sums in LDS, two sets in turn: one is read
                // while the next base row's are written
                float* set = red + (phase & 1) * (kTrWaves * NV);
                if ((tid & 63) < 4) {
#pragma unroll
                    for (int i = 0; i < NV / 4; ++i) set[(tid >> 6) * NV + 4 * i + (tid & 3)] = sum[i];
                }
                __syncthreads();
                if (tid < 2 * DC) {
                    float total = 0.0f;
                    for (int i = 0; i < TB / 64; ++i) total += set[i * NV + tid];
                    part[tid] = total;
                }
            } else {
                part += (tid >> 6) * (kNJ * DC * 2);
                if ((tid & 63) < 4) {
#pragma unroll
                    for (int i = 0; i < NV / 4; ++i)
                        if (4 * i + (tid & 3) < 2 * DC) part[4 * i + (tid & 3)] = sum[i];
                }
                __syncthreads();
            }
            ++phase;
        }
        cur = next;
    }
}

// grad[t][b] = sum over the frames, in a fixed order; grid (blocks, T).
__global__ void __launch_bounds__(256) train_grad_kernel(const TrainArgs A, int blocks, float* grad) {
    __shared__ float sw[256], sb[256];
    const int b = blockIdx.x, t = blockIdx.y;
    const float2* part = reinterpret_cast<const float2*>(A.gpart) + (size_t)t * A.gamma * A.parts * blocks + b;
    float aw = 0.0f, ab = 0.0f;
    for (int i = threadIdx.x; i < A.gamma * A.parts; i += 256) {
        const float2 v = part[(size_t)i * blocks];
        aw += v.x;
        ab += v.y;
    }
    sw[threadIdx.x] = aw;
    sb[threadIdx.x] = ab;
    __syncthreads();
    for (int h = 128; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) {
            sw[threadIdx.x] += sw[threadIdx.x + h];
            sb[threadIdx.x] += sb[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        grad[((size_t)t * blocks + b) * 2 + 0] = sw[0];
        grad[((size_t)t * blocks + b) * 2 + 1] = sb[0];
    }
}

__global__ void __launch_bounds__(256) train_loss_kernel(const TrainArgs A, float* loss) {
    __shared__ float sl[256];
    float a = 0.0f;
    for (int i = threadIdx.x; i < A.gamma; i += 256) a += A.lpart[(size_t)blockIdx.x * A.gamma + i];
    sl[threadIdx.x] = a;
    __syncthreads();
    for (int h = 128; h >= 1; h >>= 1) {
        if ((int)threadIdx.x < h) sl[threadIdx.x] += sl[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[blockIdx.x] = sl[0] * A.inv_count;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

namespace {

struct TrainVariant {
    int nj, nq, dc, maxt;
    const void *forward, *backward[2];   // backward: one sum per wavefront (few of them), per frame
};

template <int NQ, int DC>
constexpr TrainVariant train() {
    return TrainVariant{3, NQ, DC, 1024, reinterpret_cast<const void*>(&train_forward_kernel<NQ, DC>),
                        {reinterpret_cast<const void*>(&train_backward_kernel<3, NQ, DC, 1024, (NQ > 1)>),
                         reinterpret_cast<const void*>(&train_backward_kernel<3, NQ, DC, 1024, true>)}};
}
template <int DC, int MAXT>
constexpr TrainVariant train4() {
    return TrainVariant{4, 1, DC, MAXT, reinterpret_cast<const void*>(&train_forward4_kernel<DC, MAXT>),
                        {reinterpret_cast<const void*>(&train_backward_kernel<4, 1, DC, MAXT, (MAXT > 512)>),
                         reinterpret_cast<const void*>(&train_backward_kernel<4, 1, DC, MAXT, true>)}};
}

// 54 edges per thread at most; of 4-row bases 96, with fewer threads and more
// registers for each
const TrainVariant kTrain[] = {train<1, 6>(), train<2, 6>(), train<3, 6>(), train<1, 9>(),
                               train<2, 9>(), train<1, 18>(), train4<24, 512>(), train4<24, 768>()};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// two arrays by place, then the loss sums, or the shifts and two sets of sums
// per wavefront
size_t lds_bytes(const QCDesc& D) {
    return (2 * (size_t)D.n + kTrRows * kTrSlots + 2 * kTrWaves * 2 * kTrSlots) * sizeof(float);
}

const TrainVariant* covered(const ldpc_graph* g) {
    const QCDesc& D = g->qc;
    if (g->kind != LDPC_GRAPH_QC) return nullptr;
    for (int j = 0; j < D.J; ++j)
        if (D.rstart[j + 1] - D.rstart[j] != D.L) return nullptr;   // a zero block
    int dev = 0, limit = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&limit, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) {
        (void)hipGetLastError();
        limit = 160 * 1024;   // sizing without a device (gfx950's LDS)
    }
    if (lds_bytes(D) > (size_t)limit) return nullptr;
    for (const TrainVariant& v : kTrain)
        if (v.nj == D.J && v.dc == D.L && (D.p + v.nq - 1) / v.nq <= v.maxt) return &v;
    return nullptr;
}

struct TrainSpace {
    size_t rows, post, lpart, gpart, total;
};

int threads(const TrainVariant& v, const QCDesc& D) { return ((D.p + v.nq - 1) / v.nq + 63) / 64 * 64; }

// Partial sums of a frame's weight gradients.  One for each wavefront leaves
// the sum over wavefronts out of the workgroup's chain of steps; one for the
// frame saves their bytes, which count with many wavefronts.  3 x 6, p = 3060,
// 1024 frames (16 wavefronts) 1715 and 1621 us for the step; 4 x 24, p = 194, 22
// frames (4) 533 and 545.
int parts(const TrainVariant& v, const QCDesc& D) { return threads(v, D) >= 512 ? 1 : threads(v, D) / 64; }

TrainSpace train_space(const TrainVariant& v, const QCDesc& D, int gamma, int T) {
    TrainSpace S{};
    size_t off = 0;
    auto take = [&](size_t floats) { size_t o = off; off = align256(off + floats * sizeof(float)); return o; };
    S.rows = take((size_t)gamma * T * tr_words(v.dc) * D.J * D.p);
    S.post = take((size_t)gamma * T * D.n);
    S.lpart = take((size_t)gamma * T);
    S.gpart = take((size_t)gamma * T * parts(v, D) * D.nb * 2);
    S.total = off;
    return S;
}

TrainArgs train_args(const TrainVariant& v, const ldpc_graph* g, int gamma, int T, const float* w, void* ws) {
    const QCDesc& D = g->qc;
    const TrainSpace S = train_space(v, D, gamma, T);
    char* base = reinterpret_cast<char*>(ws);
    TrainArgs A{};
    A.w = w;
    A.rows = reinterpret_cast<float*>(base + S.rows);
    A.post = reinterpret_cast<float*>(base + S.post);
    A.lpart = reinterpret_cast<float*>(base + S.lpart);
    A.gpart = reinterpret_cast<float*>(base + S.gpart);
    A.inv_count = (float)(1.0 / ((double)gamma * D.n));
    A.n = D.n;
    A.p = D.p;
    A.T = T;
    A.gamma = gamma;
    A.parts = parts(v, D);
    for (int j = 0; j < D.J; ++j)
        for (int k = 0; k < D.L; ++k)
            A.sh4[j * kTrSlots + k] = 4u * (uint32_t)((D.eshift[D.rstart[j] + k] - D.eshift[k] + D.p) % D.p);
    for (int k = 0; k < D.L; ++k) A.rot4[k] = 4u * (uint32_t)D.eshift[k];
    return A;
}

bool launch(const void* fn, const ldpc_graph* g, const TrainVariant& v, TrainArgs& A, hipStream_t st) {
    const size_t lds = lds_bytes(g->qc);
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) return false;
    void* args[] = {&A};
    return hipLaunchKernel(fn, dim3((unsigned)A.gamma), dim3((unsigned)threads(v, g->qc)), args, lds, st) == hipSuccess;
}

}  // namespace

size_t train_onchip_bytes(const ldpc_graph* g, int gamma, int T) {
    const TrainVariant* v = covered(g);
    return v ? train_space(*v, g->qc, gamma, T).total : 0;
}

bool train_onchip_forward(const ldpc_graph* g, const float* llr, int gamma, int T, const float* w, float* loss,
                          void* ws, hipStream_t st) {
    const TrainVariant* v = covered(g);
    if (!v) return false;
    TrainArgs A = train_args(*v, g, gamma, T, w, ws);
    A.llr = llr;
    {
        timing::Scope ts(12, st);
        if (!launch(v->forward, g, *v, A, st)) return false;
    }
    timing::Scope ts(16, st);
    train_loss_kernel<<<(unsigned)T, 256, 0, st>>>(A, loss);
    return hipGetLastError() == hipSuccess;
}

bool train_onchip_backward(const ldpc_graph* g, int gamma, int T, const float* w, const float* dloss, float* grad,
                           void* ws, hipStream_t st) {
    const TrainVariant* v = covered(g);
    if (!v) return false;
    TrainArgs A = train_args(*v, g, gamma, T, w, ws);
    A.dloss = dloss;
    {
        timing::Scope ts(15, st);
        if (!launch(v->backward[A.parts == 1 && threads(*v, g->qc) > 64 ? 1 : 0], g, *v, A, st)) return false;
    }
    timing::Scope ts(16, st);
    train_grad_kernel<<<dim3((unsigned)g->qc.nb, (unsigned)T), 256, 0, st>>>(A, g->qc.nb, grad);
    return hipGetLastError() == hipSuccess;
}

}  // namespace ldpc
