// Block decoder with a whole frame on one compute unit (gfx950), for codes
// whose posterior sums are too large, or whose check rows are too heavy, for
// the kernel of onchip.hip: the rate-5/6 4 x 24 codes up to n = 24,576, for
// instance (their learned min-sum: onchip_nms.hip).  As there, one workgroup decodes one frame, thread i keeps the
// check-to-variable messages of check rows (j, i + q*TB) of every base row in
// registers for the whole decode, and beta = clip(L - alpha) is formed from
// the posterior sums in LDS.  What differs:
//
//   * One sum per variable instead of two.  An iteration first updates all
//     check rows from the sums (every thread, all base rows, no barrier in
//     between), then, base row by base row with a barrier after each, adds
//     the new messages into the sums.  n floats of LDS (two arrays of n would
//     not fit), at J + 2 barriers per iteration (J + 3 with
//     early stopping) instead of J.
//   * Addresses without a wrap.  The rows of a wavefront are consecutive, so
//     the variables an edge slot meets are consecutive in a base column up to
//     one wrap.  Every column is stored with 64 further cells behind its p
//     sums, so a wavefront's 64 variables are one run of cells, whose first
//     cell one lane holds for all: one vector operation per edge.  While
//     sums are accumulated, a further cell takes the part of its variable's
//     sum that arrives across the wrap; a last short step adds the two parts
//     and writes the total to both.
//   * Posteriors from the messages alone: mu + ln 2 (sum of the alphas), the
//     sums formed once more at the end without mu.  Taken from the sums in
//     LDS, whose rounding is that of the whole of L, the posteriors' error
//     against 64 bits was up to 1.24 times the package decoder's, now
//     0.93-1.01 times.  So the alphas must still be there when a frame stops:
//     the syndrome is tested in a pass of its own over the signs of the sums,
//     before the next update (which a decoded frame then saves); a wavefront
//     leaves the pass at its first base row that is violated, the first of
//     all while a frame is far from decoded.  4 x 24, early stopping, sums in
//     LDS and no such pass / this: p = 422, 1024 frames 155 / 155 us where
//     they decode, 1149 / 1196 (1409 over all rows) where none does in 30
//     iterations; p = 81, 300 frames 37 / 41; without early stopping 2 %.
//   * Row updates in place and in blocks: a row's inputs replace its old
//     messages, and the sweeps of Eq. 3 keep suffix pairs of one block of
//     slots at a time (check2e_row), so that the 96 messages of four rows of
//     weight 24 and their update fit the 128 registers a thread has with four
//     wavefronts on a SIMD.
//
// The decode is bound by the vector ALUs: about 22 plain instructions and 3
// transcendentals per edge and iteration (counted; the ALUs are busy 85 % of
// the time).  4 x 24 code, p = 1024, 1024 frames, 30 iterations: 2.50 ms
// (98,304 edges per frame: 1.21 10^12 edge updates per second), 12.15 ms with
// the message-package decoder, which streams every message through HBM twice
// an iteration.  Tried on the way
// there: (u, w, s) triples instead of pairs, two rows per thread, 512 threads
// and run bases formed by the scalar unit 3.9 ms.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>

#include "check2.h"
#include "device.h"
#include "internal.h"
#include "onchip.h"

namespace ldpc {

constexpr int kOwRows = 4;     // base rows an instantiation may have
constexpr int kOwSlots = 24;   // edge slots per row an instantiation may have
constexpr int kOwPad = 64;     // further cells behind each column
constexpr int kOwMinP = 64;    // a further cell repeats a cell of its own column

// Edge slot k of base row j (index j * kOwSlots + k): row (j, s) meets
// variable (k, (s + a) mod p) of base column k.  Byte offsets.
struct WideEdge {
    uint32_t sh4;     // 4 a
    uint32_t cb4;     // 4 k (p + kOwPad): the column's first cell
    uint32_t gb4;     // 4 k p: the column's first channel LLR
};

struct WideArgs {
    WideEdge e[kOwRows * kOwSlots];
    const float* llr;                 // [gamma][n]
    float* post;                      // [gamma][n]
    uint8_t* bits;                    // [gamma][n]
    int32_t* iters;                   // [gamma] or NULL
    uint8_t* conv;                    // [gamma] or NULL
    int32_t n, p, L, max_iters;
};

__device__ __forceinline__ float* ow_cell(float* L, uint32_t byte) {
    return reinterpret_cast<float*>(reinterpret_cast<char*>(L) + byte);
}

// One frame per workgroup.  NJ base rows, NQ rows per thread and base row, DC
// slots per row (the base is full: DC columns, DC blocks in every row); NB:
// blocks of check2e_row; MAXT: threads
// the register budget is for; EARLY: with early stopping.
template <int NJ, int NQ, int DC, int NB, int MAXT, bool EARLY>
__global__ void __launch_bounds__(MAXT) onchip_wide_kernel(const WideArgs A) {
    // dynamic LDS: L columns of p + kOwPad sums, then two flag words
    extern __shared__ float cells[];
    const int p = A.p, nl = A.L;
    const int stride = p + kOwPad;
    uint32_t* flag = reinterpret_cast<uint32_t*>(cells + (size_t)nl * stride);
    const int tid = threadIdx.x;
    const int TB = blockDim.x;
    const size_t f0 = (size_t)blockIdx.x * A.n;
    const char* __restrict__ mu = reinterpret_cast<const char*>(A.llr + f0);
    const uint32_t p4 = 4u * (uint32_t)p, lane4 = 4u * (uint32_t)(tid & 63);
    // L of "iteration 0" is mu, so that iteration 1 reads beta = clip(mu - 0)
    // (a full base has DC columns; a group of columns' loads go out together)
    constexpr int G = DC % 8 == 0 ? 8 : 9;
    for (int t = tid; t < stride; t += TB) {
        const float* at = A.llr + f0 + (t < p ? t : t - p);
#pragma unroll 1
        for (int l0 = 0; l0 < DC; l0 += G) {
            float m[G];
#pragma unroll
            for (int i = 0; i < G; ++i) m[i] = at[(size_t)(l0 + i) * p];
#pragma unroll
            for (int i = 0; i < G; ++i) cells[(l0 + i) * stride + t] = m[i] * kLog2eF + 0.0f;
        }
    }
    if (tid < 2) flag[tid] = 0u;
    float al[NJ][NQ][DC];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int k = 0; k < DC; ++k) al[j][q][k] = 0.0f;
    __syncthreads();

    // First cell of edge slot k of this wavefront's rows (j, q): a run of 64
    // cells serves all lanes.  Lane i of run[v] holds the first cell of edge
    // 64 v + i, edges numbered (j * NQ + q) * DC + k.
    constexpr int kEdges = NJ * NQ * DC, kRuns = (kEdges + 63) / 64;
    uint32_t run[kRuns];
#pragma unroll
    for (int v = 0; v < kRuns; ++v) {
        const int i = min(v * 64 + (tid & 63), kEdges - 1);
        const int jq = i / DC;
        const WideEdge& e = A.e[(jq / NQ) * kOwSlots + i - jq * DC];
        const uint32_t t = 4u * (uint32_t)((tid & ~63) + (jq % NQ) * TB) + e.sh4;
        run[v] = e.cb4 + min(t, t - p4);
    }
    const uint32_t tid4 = 4u * (uint32_t)tid;

    // each iteration: rows, sums, syndrome; at the end (out) the sums once
    // more, of the alphas alone
    int it = 1, violated = 0;
    bool out = false;
    for (;;) {
        // opaque, so that the runs' first cells are read from the lanes where
        // they are used and not held in scalar registers (there are too few)
#pragma unroll
        for (int v = 0; v < kRuns; ++v) asm volatile("" : "+v"(run[v]));
        auto first_cell = [&](int j, int q, int k) -> uint32_t {
            const int i = (j * NQ + q) * DC + k;
            return (uint32_t)__builtin_amdgcn_readlane((int)run[i >> 6], i & 63);
        };

        // check rows: new messages from the sums of the previous iteration
        if (!out) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    if (tid4 + 4u * (uint32_t)(q * TB) < p4) {
                        float (&x)[DC] = al[j][q];
#pragma unroll
                        for (int k = 0; k < DC; ++k) {
                            const float L = *ow_cell(cells, first_cell(j, q, k) + lane4);
                            x[k] = clip2(L - x[k]);
                        }
                        check2e_row<DC, NB>(x, DC);
                    }
                }
            }
        }
        __syncthreads();

        // sums, base row by base row (within one, no two threads meet the
        // same variable, and no two lanes the same cell)
        if (tid == 0) flag[(it + 1) & 1] = 0u;
        for (int i = tid; i < nl * kOwPad; i += TB) cells[(i / kOwPad) * stride + p + i % kOwPad] = 0.0f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                if (tid4 + 4u * (uint32_t)(q * TB) < p4) {
                    constexpr int B = DC % 8 == 0 ? 8 : DC % 6 == 0 ? 6 : 9;
#pragma unroll
                    for (int k0 = 0; k0 < DC; k0 += B) {
                        // all reads of a group before its writes: the compiler cannot
                        // know that the cells differ
                        float v[B];
                        uint32_t at[B];
                        if (j == 0) {
                            // the sum starts from mu, in the variable's own cell
                            uint32_t t[B];
#pragma unroll
                            for (int i = 0; i < B; ++i) {
                                const int jk = j * kOwSlots + k0 + i;
                                t[i] = first_cell(j, q, k0 + i) + lane4 - A.e[jk].cb4;
                                t[i] = min(t[i], t[i] - p4);
                                at[i] = A.e[jk].cb4 + t[i];
                                v[i] = 0.0f;
                            }
                            if (!out) {
#pragma unroll
                                for (int i = 0; i < B; ++i)   // + 0: no -0
                                    v[i] = *reinterpret_cast<const float*>(mu + (A.e[j * kOwSlots + k0 + i].gb4 + t[i])) +
                                           0.0f;
                            }
                        } else {
#pragma unroll
                            for (int i = 0; i < B; ++i) {
                                at[i] = first_cell(j, q, k0 + i) + lane4;
                                v[i] = *ow_cell(cells, at[i]);
                            }
                        }
#pragma unroll
                        for (int i = 0; i < B; ++i) {
                            const float x = al[j][q][k0 + i];
                            *ow_cell(cells, at[i]) = j == 0 ? fmaf(v[i], kLog2eF, x) : v[i] + x;
                        }
                    }
                }
            }
            __syncthreads();
        }
        // the parts of a sum on either side of the wrap
        for (int i = tid; i < nl * kOwPad; i += TB) {
            float* c = cells + (i / kOwPad) * stride + i % kOwPad;
            const float L = c[0] + c[p];
            c[0] = L;
            c[p] = L;
        }
        __syncthreads();
        if (out) break;
        if (!EARLY && it < A.max_iters) {
            ++it;
            continue;
        }

        // the syndrome: a row's parity from the sums' sign bits (a sum is
        // never -0: it starts from mu + 0)
#pragma unroll
        for (int v = 0; v < kRuns; ++v) asm volatile("" : "+v"(run[v]));
        uint64_t viol = 0;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                if (viol != 0ull) continue;   // the wavefront has its answer
                uint32_t sx = 0;
                if (tid4 + 4u * (uint32_t)(q * TB) < p4) {
#pragma unroll
                    for (int k = 0; k < DC; ++k)
                        sx ^= __float_as_uint(*ow_cell(cells, first_cell(j, q, k) + lane4));
                }
                viol = __ballot((int32_t)sx < 0);
            }
        }
        if (viol != 0ull && (tid & 63) == 0) flag[it & 1] = 1u;
        __syncthreads();
        violated = flag[it & 1] != 0u;
        if (it < A.max_iters && violated) {
            ++it;
            continue;
        }
        out = true;
        // decisions: the sums' signs
        uint32_t first = (uint32_t)tid;
        asm volatile("" : "+v"(first));   // nothing of this is worked out ahead and held
        for (int t = (int)first; t < p; t += TB)
#pragma unroll 1
            for (int l = 0; l < DC; ++l)
                A.bits[f0 + (size_t)l * p + t] = (uint8_t)(__float_as_uint(cells[l * stride + t]) >> 31);
    }

    uint32_t first = (uint32_t)tid;
    asm volatile("" : "+v"(first));
    for (int t = (int)first; t < p; t += TB)
#pragma unroll 1
        for (int l0 = 0; l0 < DC; l0 += G) {
            float m[G];
            uint32_t neg[G];
#pragma unroll
            for (int i = 0; i < G; ++i) {
                const size_t v = f0 + (size_t)(l0 + i) * p + t;
                m[i] = A.llr[v];
                neg[i] = (uint32_t)A.bits[v] << 31;   // this thread's own store
            }
#pragma unroll
            for (int i = 0; i < G; ++i) {
                const float x = clip30(posterior2(cells[(l0 + i) * stride + t], m[i]));
                A.post[f0 + (size_t)(l0 + i) * p + t] = __uint_as_float((__float_as_uint(x) & 0x7fffffffu) | neg[i]);
            }
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

struct WideVariant {
    int nj, nq, dc, maxt;
    const void* fn;         // without early stopping
    const void* fn_early;   // with early stopping
};

template <int NJ, int NQ, int DC, int NB, int MAXT>
constexpr WideVariant wide() {
    return WideVariant{NJ, NQ, DC, MAXT,
                       reinterpret_cast<const void*>(&onchip_wide_kernel<NJ, NQ, DC, NB, MAXT, false>),
                       reinterpret_cast<const void*>(&onchip_wide_kernel<NJ, NQ, DC, NB, MAXT, true>)};
}

const WideVariant kWide[] = {
    wide<4, 1, 24, 3, 1024>(), wide<3, 1, 18, 2, 1024>(), wide<3, 2, 18, 2, 768>(), wide<3, 3, 9, 1, 1024>(),
};

// Which codes: regular bases with a base row that fills a wavefront at least
// (kOwMinP), whose rows, threads and LDS an instantiation covers.  There is no
// smallest batch: at 20 iterations a single frame takes 0.64-0.78 of the
// package decoder's time (4 x 24, p = 1024: 410 us against 526; 3 x 18, p =
// 1365: 355 against 482), 256 frames 0.24-0.3 (423 us against 1649).
struct WideChoice {
    const WideVariant* v;
    int tb;
    size_t lds;
};

bool choose_wide(const ldpc_graph* g, WideChoice& c) {
    if (!g || g->kind != LDPC_GRAPH_QC) return false;
    const QCDesc& D = g->qc;
    if (D.J > kOwRows || D.dc_max > kOwSlots || D.p < kOwMinP) return false;
    for (int j = 0; j < D.J; ++j)
        if (D.rstart[j + 1] - D.rstart[j] != D.L) return false;   // a zero block
    int dev = 0, limit = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&limit, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    const size_t lds = ((size_t)D.L * (D.p + kOwPad) + 2) * sizeof(float);
    if (lds > (size_t)limit) return false;
    for (const WideVariant& v : kWide) {
        if (v.nj != D.J || v.dc != D.dc_max) continue;
        const int per = (D.p + v.nq - 1) / v.nq;
        const int tb = (per + 63) / 64 * 64;
        if (tb > v.maxt) continue;
        c.v = &v;
        c.tb = tb;
        c.lds = lds;
        return true;
    }
    return false;
}

}  // namespace

bool onchip_wide_fits(const ldpc_graph* g) {
    WideChoice c;
    return choose_wide(g, c);
}

int onchip_wide_decode(const ldpc_graph* g, const float* llr, int gamma, int max_iters, int early, float* post,
                       uint8_t* bits, int32_t* iters, uint8_t* converged, hipStream_t st, const float* nms_w) {
    if (nms_w) return onchip_nms_decode(g, llr, gamma, max_iters, early, post, bits, iters, converged, st, nms_w);
    WideChoice c;
    if (!choose_wide(g, c)) return 0;
    const QCDesc& D = g->qc;
    WideArgs A{};
    A.llr = llr;
    A.post = post;
    A.bits = bits;
    A.iters = iters;
    A.conv = converged;
    A.n = D.n;
    A.p = D.p;
    A.L = D.L;
    A.max_iters = max_iters;
    for (int j = 0; j < D.J; ++j) {
        for (int k = 0; k < D.dc_max; ++k) {
            const int b = D.rstart[j] + k, l = D.ecol[b];
            WideEdge& e = A.e[j * kOwSlots + k];
            e.sh4 = 4u * (uint32_t)D.eshift[b];
            e.cb4 = 4u * (uint32_t)(l * (D.p + kOwPad));
            e.gb4 = 4u * (uint32_t)(l * D.p);
        }
    }
    const void* fn = early ? c.v->fn_early : c.v->fn;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)c.lds) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    timing::Scope ts(23, st);
    void* args[] = {&A};
    return hipLaunchKernel(fn, dim3((unsigned)gamma), dim3((unsigned)c.tb), args, c.lds, st) == hipSuccess ? 1 : -1;
}

}  // namespace ldpc
