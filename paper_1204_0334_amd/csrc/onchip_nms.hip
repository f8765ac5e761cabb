// Learned min-sum block decoder with a frame on one compute unit (gfx950), for
// the codes that onchip_wide.hip takes for sum-product: full bases of 4 rows of
// weight 24, or of 3 rows of weight 18 or 9, with n floats in LDS.
//
// The learned rule has no exponentials to round, so whole decodes are as exact
// as their sums: with one sum L per variable and beta = L - alpha the error
// against 64 bits was 1.17-1.2 times the message packages' in natural units,
// 1.45 in base-2 units.  Here a beta is mu + (pre + suf) as there, in the same
// order, and the results are the packages' bit for bit.
//
// One cell per variable carries the sums along the base rows: upwards from the
// last row the suffixes, then downwards the prefixes.  Row j takes its suffix
// from the cell and adds its alpha; on the way back it takes its prefix, which
// completes its beta, and adds its alpha again; the last row completes L.  2 J -
// 2 barriers per iteration (with early stopping 2 J).  A thread owns the check
// rows (j, i + q*TB) and keeps three words of each, from which the alphas are
// formed again where they are used: the two smallest magnitudes, and which edge
// holds the smallest beside the output signs.  Betas go straight into the next
// three words; only the suffixes of the base rows in between lie in registers.
// mu is read from the caller's frame, which stays in L2.
//
// Bound by the vector ALUs: 35 instructions per edge and iteration (4 x 24, p =
// 1024, counted; the ALUs are busy 82 % of the time), since an edge's address and
// its alpha are worked out again at every use.  13 iterations, packages / one sum L / here:
// 4 x 24, p = 1024, 500 frames 2.00 / 0.446 / 0.629 ms; 3 x 18, p = 1500, 400
// frames 1.59 / 0.376 / 0.419; 3 x 9, p = 2500, 300 frames 0.993 / 0.308 / 0.310.
#include <hip/hip_runtime.h>

#include "check2.h"
#include "device.h"
#include "internal.h"
#include "onchip.h"

namespace ldpc {

constexpr int kOnRows = 4, kOnSlots = 24;

struct NmsArgs {
    const float* llr;      // [gamma][n]
    float* post;           // [gamma][n]
    uint8_t* bits;         // [gamma][n]
    int32_t* iters;        // [gamma] or NULL
    uint8_t* conv;         // [gamma] or NULL
    const float* w;        // [iters][blocks][2]: (scale, offset)
    int32_t n, p, max_iters;
    uint32_t sh4[kOnRows * kOnSlots];   // 4 times the shift of edge slot k of base row j
};

// The weights: the kernel does not write them, so they are read by the scalar unit.
typedef const __attribute__((address_space(4))) float* on_weights;

// A check row's outputs: the two smallest input magnitudes, and a word of the
// output signs (slot k's in bit DC - 1 - k) and the slot of the smallest (from
// bit 24).
template <int DC>
struct NmsRow {
    float m1, m2;
    uint32_t word;

    // slot of the smallest, opaque: alphas are formed again at every use, and
    // compared with k as it stands (a comparison of a byte of the word would
    // hold each k in a register)
    __device__ __forceinline__ uint32_t smallest() {
        asm volatile("" : "+v"(m1), "+v"(word));
        uint32_t i = word >> 24;
        asm volatile("" : "+v"(i));
        return i;
    }
    __device__ __forceinline__ float alpha(int k, uint32_t smallest, on_weights w) const {
        const float v = fmaxf((smallest == (uint32_t)k ? m2 : m1) - w[2 * k + 1], 0.0f);
        // rounded before it is added to a sum
        {
#pragma clang fp contract(off)
            return w[2 * k] * __builtin_copysignf(v, __uint_as_float(word << (32 - DC + k)));
        }
    }
};

// The same while a row's inputs come, slot by slot.
template <int DC>
struct NmsInputs {
    float m1 = __builtin_inff(), m2 = __builtin_inff();
    uint32_t sgn = 0, i1 = 0;

    __device__ __forceinline__ void add(int k, float x) {
        const float m = fabsf(x);
        sgn = __builtin_amdgcn_alignbit(sgn, __float_as_uint(x), 31);
        m2 = __builtin_amdgcn_fmed3f(m, m1, m2);
        i1 = m < m1 ? (uint32_t)k : i1;
        m1 = fminf(m, m1);
    }
    __device__ __forceinline__ NmsRow<DC> row() const {
        const uint32_t s = sgn ^ (0u - ((uint32_t)__builtin_popcount(sgn) & 1u));
        return NmsRow<DC>{m1, m2, (s & ((1u << DC) - 1u)) | i1 << 24};
    }
};

__device__ __forceinline__ float* on_at(float* base, uint32_t byte) {
    return reinterpret_cast<float*>(reinterpret_cast<char*>(base) + byte);
}

// NJ base rows, NQ rows per thread and base row, DC slots per row; MAXT: threads
// the register budget is for; KEEP: the alphas of the base rows in between lie
// in registers too; EARLY: with early stopping.
template <int NJ, int NQ, int DC, int MAXT, bool KEEP, bool EARLY>
__global__ void __launch_bounds__(MAXT) onchip_nms_kernel(const NmsArgs A) {
    extern __shared__ float cells[];   // [n], then two flag words
    const int n = A.n, p = A.p, tid = threadIdx.x, TB = blockDim.x;
    uint32_t* flag = reinterpret_cast<uint32_t*>(cells + n);
    const uint32_t p4 = 4u * (uint32_t)p, TB4 = 4u * (uint32_t)TB;
    const size_t f0 = (size_t)blockIdx.x * n;
    const char* __restrict__ mu = reinterpret_cast<const char*>(A.llr + f0);
    constexpr int B = DC == 24 ? 4 : DC == 18 && NQ == 1 ? 6 : 3;   // edges whose reads go out together

    NmsRow<DC> row[NJ][NQ];
    float suf[NJ - 2][NQ][DC];   // suffixes of the rows in between
    float al[KEEP ? NJ - 2 : 1][KEEP ? NQ : 1][KEEP ? DC : 1];   // their alphas
    uint32_t tid4 = 4u * (uint32_t)tid;
    // byte of the variable that slot k of row (j, s) meets
    auto var = [&](int j, int k, uint32_t s4) -> uint32_t {
        const uint32_t t = s4 + A.sh4[j * kOnSlots + k];
        return (uint32_t)k * p4 + min(t, t - p4);
    };
    // each row of base row j, its edges in groups: act(q, k, the row's smallest,
    // the cell's byte, its value, mu) for the edges of a group after all their
    // reads, then done(q)
    auto each = [&](int j, bool read, bool with_mu, auto&& act, auto&& done) {
        asm volatile("" : "+v"(tid4));   // offsets are worked out again at every step, not held
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const uint32_t s4 = tid4 + (uint32_t)q * TB4;
            if (s4 < p4) {
                const uint32_t i1 = row[j][q].smallest();
#pragma unroll
                for (int k0 = 0; k0 < DC; k0 += B) {
                    uint32_t at[B];
                    float v[B], m[B];
#pragma unroll
                    for (int i = 0; i < B; ++i) {
                        at[i] = var(j, k0 + i, s4);
                        v[i] = read ? *on_at(cells, at[i]) : 0.0f;
                        m[i] = with_mu ? *reinterpret_cast<const float*>(mu + at[i]) : 0.0f;
                    }
#pragma unroll
                    for (int i = 0; i < B; ++i) act(q, k0 + i, i1, at[i], v[i], m[i]);
                }
                done(q);
            }
        }
    };
    auto nothing = [](int) {};
    NmsInputs<DC> in[NQ];
    auto take = [&](int j) {
        return [&, j](int q) {
            row[j][q] = in[q].row();
            in[q] = NmsInputs<DC>{};
        };
    };

    // the first messages are the channel LLRs
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) row[j][q] = NmsRow<DC>{0.0f, 0.0f, 0u};
        each(j, false, true, [&](int q, int k, uint32_t, uint32_t, float, float m) {
            const float c = fminf(fabsf(m), kClip);
            in[q].add(k, m < 0.0f ? -c : c);
        }, take(j));
    }
#pragma unroll
    for (int j = 0; j < NJ - 2; ++j)
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int k = 0; k < DC; ++k) {
                suf[j][q][k] = 0.0f;
                if (KEEP) al[KEEP ? j : 0][KEEP ? q : 0][KEEP ? k : 0] = 0.0f;
            }
    if (tid < 2) flag[tid] = 0u;

    int it = 1;
    bool violated;
    auto weights = [&](int j) { return (on_weights)(uintptr_t)A.w + ((size_t)(it - 1) * NJ + j) * (DC * 2); };
    // from the last base row's prefixes L, in the cells, and its betas; whether
    // a row is violated by L's decisions
    auto complete = [&]() -> bool {
        const on_weights w = weights(NJ - 1);
        uint32_t odd[NQ];   // parity of a row's decisions
#pragma unroll
        for (int q = 0; q < NQ; ++q) odd[q] = 0u;
        each(NJ - 1, true, true, [&](int q, int k, uint32_t i1, uint32_t at, float v, float m) {
            in[q].add(k, clip30(m + v));
            const float L = m + (v + row[NJ - 1][q].alpha(k, i1, w));
            *on_at(cells, at) = L;
            odd[q] ^= (uint32_t)(L < 0.0f);
        }, take(NJ - 1));
        if (tid == 0) flag[(it + 1) & 1] = 0u;
        __syncthreads();
        uint64_t viol = 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) viol |= __ballot(odd[q] != 0u);
#pragma unroll
        for (int j = 0; j < NJ - 1; ++j) {
            if (viol != 0ull) continue;   // the wavefront has its answer
#pragma unroll
            for (int q = 0; q < NQ; ++q) odd[q] = 0u;
            each(j, true, false, [&](int q, int, uint32_t, uint32_t, float v, float) { odd[q] ^= (uint32_t)(v < 0.0f); },
                 nothing);
#pragma unroll
            for (int q = 0; q < NQ; ++q) viol |= __ballot(odd[q] != 0u);
        }
        if (viol != 0ull && (tid & 63) == 0) flag[it & 1] = 1u;
        __syncthreads();
        return flag[it & 1] != 0u;
    };
    for (;; ++it) {
        {
            const on_weights w = weights(NJ - 1);
            each(NJ - 1, false, false, [&](int q, int k, uint32_t i1, uint32_t at, float, float) {
                *on_at(cells, at) = 0.0f + row[NJ - 1][q].alpha(k, i1, w);
            }, nothing);
        }
        __syncthreads();
        // suffixes
#pragma unroll
        for (int j = NJ - 2; j >= 1; --j) {
            const on_weights w = weights(j);
            each(j, true, false, [&](int q, int k, uint32_t i1, uint32_t at, float v, float) {
                const float a = row[j][q].alpha(k, i1, w);
                suf[j - 1][q][k] = v;
                if (KEEP) al[KEEP ? j - 1 : 0][KEEP ? q : 0][KEEP ? k : 0] = a;
                *on_at(cells, at) = v + a;
            }, nothing);
            __syncthreads();
        }
        {
            const on_weights w = weights(0);
            each(0, true, true, [&](int q, int k, uint32_t i1, uint32_t at, float v, float m) {
                in[q].add(k, clip30(m + v));
                *on_at(cells, at) = 0.0f + row[0][q].alpha(k, i1, w);
            }, take(0));
        }
        __syncthreads();
        // prefixes
#pragma unroll
        for (int j = 1; j < NJ - 1; ++j) {
            const on_weights w = weights(j);
            each(j, true, true, [&](int q, int k, uint32_t i1, uint32_t at, float v, float m) {
                in[q].add(k, clip30(m + (v + suf[j - 1][q][k])));
                const float a = KEEP ? al[KEEP ? j - 1 : 0][KEEP ? q : 0][KEEP ? k : 0] : row[j][q].alpha(k, i1, w);
                *on_at(cells, at) = v + a;
            }, take(j));
            __syncthreads();
        }
        if constexpr (EARLY) {
            violated = complete();
            if (it == A.max_iters || !violated) break;
        } else {
            if (it == A.max_iters) break;
            // the cells are this row's own until it publishes its next alphas
            each(NJ - 1, true, true, [&](int q, int k, uint32_t, uint32_t, float v, float m) {
                in[q].add(k, clip30(m + v));
            }, take(NJ - 1));
        }
    }
    if constexpr (!EARLY) violated = complete();

    for (int v = tid; v < n; v += TB) {
        const float L = cells[v];
        A.post[f0 + v] = clip30(L);
        A.bits[f0 + v] = (uint8_t)(L < 0.0f);
    }
    if (tid == 0) {
        if (A.iters) A.iters[blockIdx.x] = it;
        if (A.conv) A.conv[blockIdx.x] = violated ? 0 : 1;
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

namespace {

struct NmsVariant {
    int nj, nq, dc, least, maxt;   // threads: at least, at most
    const void *fn, *fn_early;
};

template <int NJ, int NQ, int DC, int MAXT, bool KEEP, bool KEEP_EARLY>
constexpr NmsVariant nms(int least = 0) {
    return NmsVariant{NJ, NQ, DC, least, MAXT,
                      reinterpret_cast<const void*>(&onchip_nms_kernel<NJ, NQ, DC, MAXT, KEEP, false>),
                      reinterpret_cast<const void*>(&onchip_nms_kernel<NJ, NQ, DC, MAXT, KEEP_EARLY, true>)};
}

// The codes of onchip_wide.hip's instantiations.  The alphas of two base rows of
// weight 24 beside their suffixes leave a workgroup of up to 768 threads without
// a second one on its compute unit, and with early stopping spill: 500 frames,
// 13 iterations, kept / formed again: p = 584 429 / 494 us, with early stopping
// 228 / 176; p = 384 (two workgroups where they are not kept) 332 / 292.
const NmsVariant kNms[] = {nms<4, 1, 24, 768, true, false>(513), nms<4, 1, 24, 1024, false, false>(),
                           nms<3, 1, 18, 1024, true, true>(), nms<3, 2, 18, 768, true, true>(),
                           nms<3, 3, 9, 1024, true, true>()};

}  // namespace

int onchip_nms_decode(const ldpc_graph* g, const float* llr, int gamma, int max_iters, int early, float* post,
                      uint8_t* bits, int32_t* iters, uint8_t* converged, hipStream_t st, const float* nms_w) {
    if (!onchip_wide_fits(g)) return 0;
    const QCDesc& D = g->qc;
    const NmsVariant* v = nullptr;
    int tb = 0;
    for (const NmsVariant& c : kNms) {
        tb = ((D.p + c.nq - 1) / c.nq + 63) / 64 * 64;
        if (c.nj == D.J && c.dc == D.L && tb >= c.least && tb <= c.maxt) {
            v = &c;
            break;
        }
    }
    if (!v) return 0;
    NmsArgs A{};
    A.llr = llr;
    A.post = post;
    A.bits = bits;
    A.iters = iters;
    A.conv = converged;
    A.w = nms_w;
    A.n = D.n;
    A.p = D.p;
    A.max_iters = max_iters;
    for (int j = 0; j < D.J; ++j)
        for (int k = 0; k < D.L; ++k) A.sh4[j * kOnSlots + k] = 4u * (uint32_t)D.eshift[D.rstart[j] + k];
    const void* fn = early ? v->fn_early : v->fn;
    const size_t lds = ((size_t)D.n + 2) * sizeof(float);
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    timing::Scope ts(23, st);
    void* args[] = {&A};
    return hipLaunchKernel(fn, dim3((unsigned)gamma), dim3((unsigned)tb), args, lds, st) == hipSuccess ? 1 : -1;
}

}  // namespace ldpc
