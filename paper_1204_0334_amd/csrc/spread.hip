// Block decoder with a frame spread over several compute units (gfx950), for
// full bases of 3 rows of weight 6, 9 or 18.
//
// On one compute unit (onchip.hip) an iteration of a long code is bound by
// that unit's vector ALUs: 8 us for 3 x 6, p = 3060, with 255 of 256 units
// idle when there is one frame; longer codes do not fit one unit, and their
// message packages take two launches per iteration.  Here C workgroups share a frame: member c
// owns the check rows (j, s), c TB <= s < (c + 1) TB, one offset s per thread
// with the rows of all three base rows, and keeps their messages alpha and
// channel LLRs in registers.  Per edge a thread reads the alphas of the other
// two rows of the edge's variable, forms L = ((mu + a0) + a1) + a2 as the
// one-unit decoder's sums are formed, and beta = clip(L - own alpha): every
// row forms its variables' sums itself, so there is one exchange per
// iteration, no sum is shared, and the results are the one-unit decoder's bit
// for bit; of codes too long for one unit, in their arithmetic, the message
// packages'.
//
// The exchange needs no barrier.  An alpha travels as one 64-bit word (value,
// iteration) through device-coherent stores and loads, and a reader repeats
// its loads until the words carry the iteration it wants; nothing relies on
// the order in which two words become visible.  Two words per edge (iteration
// & 1) are enough: the thread at the other end of a variable writes its alpha
// of iteration i + 2 only after it has read the reader's alpha of i + 1 on
// the same variable, which the reader wrote after it had read the alpha of
// iteration i.  The words are cleared first, in a launch of their own: to
// alphas 0 of iteration 0.
//
// Early stopping: a member publishes whether one of its rows is violated, in
// a word of the same form, and every member reads all of them an iteration
// later, beside the alphas, when L of the iteration they speak of is still at
// hand.
//
// Every wait ends, and no result depends on how one ends.  Workgroups take
// their places in the order in which they start, so at most one frame of a
// launch has a member that has not started, and at most C - 1 workgroups wait
// for it; a device with a unit mask, or several such launches that fill an
// XCD between them, can all the same leave it without room.  So a wavefront
// tries kSpTries times (0.1 s) and then gives up: it publishes nothing more,
// writes no output, and its workgroup leaves with a mark in the frame's word
// `left`, in which all workgroups of a frame are counted as they leave.  What
// the others got was right, or they run out of tries themselves.  The last
// one to leave finds the mark and decodes the frame alone, in the same
// arithmetic, without waiting for anybody (3 x 6, p = 3060: 95 us per
// iteration).
//
// 3 x 6, p = 3060, 20 iterations with early stopping: 1 frame 85 us for 168 on
// one unit, 16 frames 124 for 169 (96 and 127 before all words of a try were
// in flight together).  An iteration of one frame takes 3 us without early
// stopping, 3.8 with, most of them the exchange.
// Codes too long for one unit, 20 iterations, spread / message packages: 3 x 6,
// p = 3600, 1 frame 101 / 434 us; 3 x 9, 16 frames 187; 3 x 18, 8 frames 236 /
// 940.  In the one-unit decoder's arithmetic they took 79, 187 and 212, but
// then a frame's results depended on the batch, and their error against 64
// bits was up to 1.2 times the packages'.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>

#include "check2.h"
#include "device.h"
#include "internal.h"
#include "onchip.h"
#include "spread.h"

namespace ldpc {

constexpr int kSpRows = 3, kSpSlots = 18, kSpMembers = 16, kSpThreads = 256;

struct SpreadArgs {
    const float* llr;      // [gamma][n]
    float* post;           // [gamma][n]
    uint8_t* bits;         // [gamma][n]
    int32_t* iters;        // [gamma] or NULL
    uint8_t* conv;         // [gamma] or NULL
    const float* nms_w;    // learned min-sum (RULE 1): [iters][blocks][2]
    uint64_t* box;         // [gamma][2][E]: alpha of edge (j DC + k) p + s, slot iteration & 1
    uint64_t* verdict;     // [gamma][2][kSpMembers]
    uint32_t* ticket;      // workgroups that have started
    uint32_t* left;        // [gamma] workgroups of the frame that have left, and from bit 16 those that gave up
    int32_t n, p, gamma, max_iters, members, nb;
    uint32_t tries;        // of a wavefront, before it gives up
    int32_t rb0[kSpRows];                      // first block of base row j
    uint32_t sh4[kSpRows * kSpSlots];          // 4 times the shift of edge slot k of base row j
    // 8 times the offset from row (j, s) to the row of base row (j + 1) % 3
    // (first) and (j + 2) % 3 (second) that meets the variable of its slot k
    uint32_t to1[kSpRows * kSpSlots], to2[kSpRows * kSpSlots];
};

// words in device memory
typedef __attribute__((address_space(1))) uint64_t sp_word;
typedef __attribute__((address_space(1))) char sp_byte;

__device__ __forceinline__ uint64_t sp_load(sp_word* base, uint32_t byte) {
    return __hip_atomic_load((sp_word*)((sp_byte*)base + byte), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void sp_store(sp_word* base, uint32_t byte, uint32_t value, uint32_t tag) {
    __hip_atomic_store((sp_word*)((sp_byte*)base + byte), (uint64_t)value | (uint64_t)tag << 32, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// RULE 0, 1: sum-product and learned min-sum as on one unit (onchip.hip), whose
// results are equal bit for bit; 2, 3: the same as in the message packages
// (natural units, a variable's beta the sum of the other alphas), with the
// results of which those of codes that no unit takes are equal bit for bit.
constexpr bool sp_packages(int rule) { return rule >= 2; }

// Channel LLR as the sums take it (on one unit no sum is ever -0).
template <int RULE>
__device__ __forceinline__ float spread_mu(float mu) {
    return sp_packages(RULE) ? mu : mu + 0.0f;
}

// Sum L of a variable, and the beta that it sends to its row of base row j;
// a: its alphas by base row (all 0 before iteration 1: first).
template <int RULE>
__device__ __forceinline__ float spread_sum(float m, const float (&a)[kSpRows], int j, bool first, float& beta) {
    if constexpr (sp_packages(RULE)) {
        const float mu[1] = {m};
        float al[kSpRows][1], b[kSpRows][1], L[1];
#pragma unroll
        for (int i = 0; i < kSpRows; ++i) al[i][0] = a[i];
        sp_variable<kSpRows, 1>(mu, al, b, L);
        // the first message is mu itself, which the rule clips
        const float c = fminf(fabsf(m), kClip), from_mu = RULE == 2 ? m : m < 0.0f ? -c : c;
        beta = first ? from_mu : j == 0 ? b[0][0] : j == 1 ? b[1][0] : b[2][0];
        return L[0];
    } else {
        const float L = (fmaf(m, kLog2eF, a[0]) + a[1]) + a[2];
        beta = clip2(L - (j == 0 ? a[0] : j == 1 ? a[1] : a[2]));
        return L;
    }
}

// What a sum adds to its row's parity, in bit 31 (on one unit no sum is ever
// -0: it starts from mu + 0).
template <int RULE>
__device__ __forceinline__ uint32_t spread_sign(float L) {
    return sp_packages(RULE) ? (L < 0.0f ? 0x80000000u : 0u) : __float_as_uint(L);
}

// The rule of base row j at iteration it, in place.
template <int DC, int RULE>
__device__ __forceinline__ void spread_rule(const SpreadArgs& A, int it, int j, float (&x)[DC]) {
    const float* w = RULE % 2 ? A.nms_w + ((size_t)(it - 1) * A.nb + A.rb0[j]) * 2 : nullptr;
    if constexpr (RULE == 0) {
        check2e_row<DC, DC <= 9 ? 1 : 2>(x, DC);
    } else if constexpr (RULE == 1) {
        nms2_row<DC>(x, DC, w, x);
    } else if constexpr (RULE == 2) {
        // sp_check, at the package kernels' row capacity (12 and 24 for rows of
        // weight 9 and 18) as far as it can be seen: whether a slot follows
        // the row's last decides how that one's output is rounded
        constexpr int N = DC == 6 ? DC : DC + 1;
        float t[N], q[N], mag[N];
        uint32_t sgn = 0;
#pragma unroll
        for (int k = 0; k < DC; ++k) {
            tq_of(x[k], t[k], q[k]);
            sgn ^= __float_as_uint(x[k]) & 0x80000000u;
        }
        if constexpr (N > DC) {
            t[DC] = 1.0f;
            q[DC] = 0.0f;
            asm volatile("" : "+v"(t[DC]), "+v"(q[DC]));
        }
        boxplus_fb<N>(t, q, mag);
#pragma unroll
        for (int k = 0; k < DC; ++k)
            x[k] = __uint_as_float(__float_as_uint(mag[k]) | (sgn ^ (__float_as_uint(x[k]) & 0x80000000u)));
    } else {
        nms2_row<DC, false>(x, DC, w, x);
    }
}

// DC: row weight; RULE as above; EARLY: with early stopping.  Two workgroups fit a compute unit (256 registers).  The words of
// all three rows are in flight together, of heavy rows those of one row.
template <int DC, int RULE, bool EARLY>
__global__ void __launch_bounds__(kSpThreads) __attribute__((amdgpu_waves_per_eu(2)))
spread_kernel(const SpreadArgs A) {
    // failed: a wavefront of this workgroup has given up
    __shared__ uint32_t place, bad[3], go, failed;
    const int tid = threadIdx.x, TB = blockDim.x, p = A.p;
    if (tid == 0) {
        place = __hip_atomic_fetch_add(A.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bad[0] = bad[1] = bad[2] = failed = 0u;
    }
    __syncthreads();
    const uint32_t me = __builtin_amdgcn_readfirstlane(place);
    const uint32_t frame = me / (uint32_t)A.members, member = me - frame * (uint32_t)A.members;
    if (frame >= (uint32_t)A.gamma) return;   // only where another launch uses the same workspace
    const size_t f0 = (size_t)frame * A.n;
    const float* __restrict__ llr = A.llr + f0;
    const uint32_t p4 = 4u * (uint32_t)p, p8 = 8u * (uint32_t)p;
    const uint32_t s = member * (uint32_t)TB + (uint32_t)tid;
    const bool active = s < (uint32_t)p;
    const uint32_t s4 = 4u * s, s8 = 8u * s;
    const size_t E = (size_t)kSpRows * DC * p;
    sp_word* const box = (sp_word*)A.box + (size_t)frame * 2 * E;
    sp_word* const verdict = (sp_word*)A.verdict + (size_t)frame * 2 * kSpMembers;
    uint32_t* const left = A.left + frame;
    uint32_t tries = A.tries;
    bool alive = true;   // this wavefront has not given up

    auto channel = [&](int j, int k, uint32_t r4) -> uint32_t {   // byte of the LLR that slot k of row (j, r) meets
        const uint32_t t = r4 + A.sh4[j * kSpSlots + k];
        return (uint32_t)k * p4 + min(t, t - p4);
    };
    auto raw = [&](int j, int k, uint32_t r4) -> float {
        return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(llr) + channel(j, k, r4));
    };
    // of heavy rows the channel LLRs are read again where they are used
    constexpr bool kMuInRegs = DC <= 9;
    float mu[kMuInRegs ? kSpRows : 1][DC], al[kSpRows][DC], Lkeep[DC];
#pragma unroll
    for (int j = 0; j < kSpRows; ++j)
#pragma unroll
        for (int k = 0; k < DC; ++k) {
            if (kMuInRegs) mu[kMuInRegs ? j : 0][k] = active ? raw(j, k, s4) : 0.0f;
            al[j][k] = 0.0f;
        }
#pragma unroll
    for (int k = 0; k < DC; ++k) Lkeep[k] = 0.0f;
    if (kMuInRegs) {
#pragma unroll
        for (int j = 0; j < kSpRows; ++j)
#pragma unroll
            for (int k = 0; k < DC; ++k) mu[kMuInRegs ? j : 0][k] = spread_mu<RULE>(mu[kMuInRegs ? j : 0][k]);
    }

    // repeats get() until no lane needs another try; false when this
    // wavefront has no tries left, or another workgroup of the frame gave up
    auto await = [&](auto&& get) -> bool {
        while (__ballot(!get()) != 0ull) {
            if (tries == 0u) return false;
            --tries;
            if ((tries & 255u) == 0u &&
                __hip_atomic_load(left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= 0x10000u)
                return false;
        }
        return true;
    };
    auto give_up = [&]() {
        alive = false;
        if ((tid & 63) == 0) failed = 1u;
    };
    // the first wavefront: whether a member's rows are violated, from the
    // words of iteration it
    auto any_violated = [&](uint32_t it) -> bool {
        bool v = false;
        if (!await([&]() -> bool {
                if (tid >= A.members) return true;
                const uint64_t w = sp_load(verdict, 8u * ((it & 1u) * kSpMembers + (uint32_t)tid));
                v = (uint32_t)w != 0u;
                return (uint32_t)(w >> 32) == it;
            }))
            give_up();
        return __ballot(v) != 0ull;
    };

    int stop = 0;
    for (int it = 1;; ++it) {
        bool fin = it > A.max_iters;
        const uint32_t want = (uint32_t)(it - 1);
        sp_word* from = box + (want & 1u) * E;
        sp_word* to = box + ((uint32_t)it & 1u) * E;
        // alphas of the other rows of the variables of rows (j, s), j0 <= j <
        // j0 + NW, iteration it - 1
        constexpr int NW = DC <= 9 ? kSpRows : 1;
        uint64_t w1[NW][DC], w2[NW][DC];
        auto fetch = [&](int j0) -> bool {
            if (!active) return true;
            // opaque: the words' offsets are worked out again at every try, not held
            uint32_t at = s8;
            asm volatile("" : "+v"(at));
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const int j = j0 + i, j1 = (j + 1) % kSpRows, j2 = (j + 2) % kSpRows;
#pragma unroll
                for (int k = 0; k < DC; ++k) {
                    const uint32_t t1 = at + A.to1[j * kSpSlots + k], t2 = at + A.to2[j * kSpSlots + k];
                    w1[i][k] = sp_load(from, (uint32_t)(j1 * DC + k) * p8 + min(t1, t1 - p8));
                    w2[i][k] = sp_load(from, (uint32_t)(j2 * DC + k) * p8 + min(t2, t2 - p8));
                }
            }
            // no load waits for the test of an earlier one
            __builtin_amdgcn_sched_barrier(0);
            uint32_t off = 0;
#pragma unroll
            for (int i = 0; i < NW; ++i)
#pragma unroll
                for (int k = 0; k < DC; ++k)
                    off |= ((uint32_t)(w1[i][k] >> 32) ^ want) | ((uint32_t)(w2[i][k] >> 32) ^ want);
            return off == 0u;
        };
        if (NW == kSpRows && alive && !await([&]() { return fetch(0); })) give_up();
        if (EARLY && it >= 3) {
            if (tid < 64) {
                const bool any = alive && any_violated(want);
                if (tid == 0) go = failed ? 2u : any ? 1u : 0u;
            }
            __syncthreads();
            const uint32_t verdict_read = go;
            if (verdict_read == 2u) {
                alive = false;
                break;
            }
            if (verdict_read == 0u) {   // the syndrome of iteration it - 2 is zero: Lkeep holds its sums
                stop = it - 2;
                break;
            }
        }
        uint64_t viol = 0;
#pragma unroll
        for (int j = 0; j < kSpRows; ++j) {
            float (&m)[DC] = mu[kMuInRegs ? j : 0];
            if (!kMuInRegs && active) {   // in flight with the words
                uint32_t at = s4;
                asm volatile("" : "+v"(at));
#pragma unroll
                for (int k = 0; k < DC; ++k) m[k] = raw(j, k, at);
            }
            if (NW == 1 && alive && !await([&]() { return fetch(j); })) give_up();
            if (!active || !alive) continue;
            if (!kMuInRegs) {
#pragma unroll
                for (int k = 0; k < DC; ++k) m[k] = spread_mu<RULE>(m[k]);
            }
            constexpr bool all = NW == kSpRows;
            float x[DC];
            uint32_t sx = 0;
#pragma unroll
            for (int k = 0; k < DC; ++k) {
                const float u = __uint_as_float((uint32_t)w1[all ? j : 0][k]);
                const float v = __uint_as_float((uint32_t)w2[all ? j : 0][k]);
                const float a[kSpRows] = {j == 0 ? al[j][k] : j == 1 ? v : u, j == 0 ? u : j == 1 ? al[j][k] : v,
                                          j == 0 ? v : j == 1 ? u : al[j][k]};
                const float L = spread_sum<RULE>(m[k], a, j, it == 1, x[k]);
                if (j == 0) Lkeep[k] = L;
                sx ^= spread_sign<RULE>(L);
            }
            viol |= __ballot((int32_t)sx < 0);
            if (!fin) {
                uint32_t at = s8;
                asm volatile("" : "+v"(at));
                spread_rule<DC, RULE>(A, it, j, x);
#pragma unroll
                for (int k = 0; k < DC; ++k) {
                    al[j][k] = x[k];
                    sp_store(to, (uint32_t)(j * DC + k) * p8 + at, __float_as_uint(x[k]), (uint32_t)it);
                }
            }
        }
        // without early stopping no other barrier comes: straight to the last
        if (!EARLY && !alive) fin = true;
        if ((EARLY && it >= 2) || fin) {
            if (viol != 0ull && (tid & 63) == 0) bad[it & 1] = 1u;
            __syncthreads();
            if (tid == 0) {
                if (!failed)
                    sp_store(verdict, 8u * (((uint32_t)it & 1u) * kSpMembers + member), bad[it & 1], (uint32_t)it);
                bad[(it + 1) & 1] = 0u;
            }
        }
        if (fin) break;
    }

    // the words are in memory before this workgroup is counted as gone
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    auto leave = [&]() -> uint32_t {
        return __hip_atomic_fetch_add(left, failed ? 0x10001u : 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const bool verdict_due = member == 0 && !stop;   // still reads the last iteration's verdicts
    uint32_t before = 0;
    if (tid == 0 && !verdict_due) before = leave();
    auto put = [&](int k, uint32_t r4, float L) {
        const size_t v = f0 + (channel(0, k, r4) >> 2);
        A.post[v] = sp_packages(RULE) ? clip30(L) : unscale2(L);
        A.bits[v] = (uint8_t)(L < 0.0f);
    };
    if (active && alive) {
#pragma unroll
        for (int k = 0; k < DC; ++k) put(k, s4, Lkeep[k]);
    }
    if (member == 0 && tid < 64) {
        const bool any = verdict_due && !failed && any_violated((uint32_t)A.max_iters + 1u);
        if (tid == 0) {
            if (!failed) {
                if (A.iters) A.iters[frame] = stop ? stop : A.max_iters;
                if (A.conv) A.conv[frame] = any ? 0 : 1;
            }
            if (verdict_due) before = leave();
        }
    }
    if (tid == 0) go = (before & 0xffffu) + 1u == (uint32_t)A.members && (before >= 0x10000u || failed) ? 1u : 0u;
    __syncthreads();
    if (go == 0u) return;

    // The last to leave a frame that a member gave up: all of its rows, one
    // iteration after the other, in the same words.
    if (tid < 3) bad[tid] = 0u;
    __syncthreads();
    for (int it = 1;; ++it) {
        const bool fin = it > A.max_iters;
        sp_word* from = box + ((uint32_t)(it - 1) & 1u) * E;
        sp_word* to = box + ((uint32_t)it & 1u) * E;
        // the sum of the variable of slot k of row (j, r) after iteration it - 1, and the beta it sends there
        auto sum = [&](int j, int k, uint32_t r, float& beta) -> float {
            const int j1 = j == 2 ? 0 : j + 1, j2 = j == 0 ? 2 : j - 1;
            const uint32_t t1 = 8u * r + A.to1[j * kSpSlots + k], t2 = 8u * r + A.to2[j * kSpSlots + k];
            float own = 0.0f, u = 0.0f, v = 0.0f;
            if (it > 1) {
                own = __uint_as_float((uint32_t)sp_load(from, (uint32_t)(j * DC + k) * p8 + 8u * r));
                u = __uint_as_float((uint32_t)sp_load(from, (uint32_t)(j1 * DC + k) * p8 + min(t1, t1 - p8)));
                v = __uint_as_float((uint32_t)sp_load(from, (uint32_t)(j2 * DC + k) * p8 + min(t2, t2 - p8)));
            }
            const float a[kSpRows] = {j == 0 ? own : j == 1 ? v : u, j == 0 ? u : j == 1 ? own : v,
                                      j == 0 ? v : j == 1 ? u : own};
            return spread_sum<RULE>(spread_mu<RULE>(raw(j, k, 4u * r)), a, j, it == 1, beta);
        };
        bool viol = false;
#pragma unroll 1
        for (uint32_t r = (uint32_t)tid; r < (uint32_t)p; r += (uint32_t)TB) {
#pragma unroll 1
            for (int j = 0; j < kSpRows; ++j) {
                float x[DC];
                uint32_t sx = 0;
#pragma unroll
                for (int k = 0; k < DC; ++k) {
                    sx ^= spread_sign<RULE>(sum(j, k, r, x[k]));
                }
                viol = viol || (int32_t)sx < 0;
                if (fin) continue;
                spread_rule<DC, RULE>(A, it, j, x);
#pragma unroll
                for (int k = 0; k < DC; ++k)
                    sp_store(to, (uint32_t)(j * DC + k) * p8 + 8u * r, __float_as_uint(x[k]), (uint32_t)it);
            }
        }
        if (viol) bad[it % 3] = 1u;
        if (tid == 0) bad[(it + 1) % 3] = 0u;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        const bool any = bad[it % 3] != 0u;
        if (!fin && !(EARLY && it >= 2 && !any)) continue;
        for (uint32_t r = (uint32_t)tid; r < (uint32_t)p; r += (uint32_t)TB)
            for (int k = 0; k < DC; ++k) {
                float beta;
                put(k, 4u * r, sum(0, k, r, beta));
            }
        if (tid == 0) {
            if (A.iters) A.iters[frame] = it - 1;
            if (A.conv) A.conv[frame] = any ? 0 : 1;
        }
        return;
    }
}

// Clears the words (count 16-byte pieces).
__global__ void __launch_bounds__(256) spread_clear_kernel(uint4* words, size_t count) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (size_t)gridDim.x * 256)
        words[i] = make_uint4(0u, 0u, 0u, 0u);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

namespace {

struct SpreadVariant {
    int dc, rule;
    const void *fn, *fn_early;
};

template <int DC, int RULE>
constexpr SpreadVariant spread() {
    return SpreadVariant{DC, RULE, reinterpret_cast<const void*>(&spread_kernel<DC, RULE, false>),
                         reinterpret_cast<const void*>(&spread_kernel<DC, RULE, true>)};
}

const SpreadVariant kSpread[] = {spread<6, 0>(), spread<9, 0>(), spread<6, 1>(), spread<9, 1>(),
                                 spread<6, 2>(), spread<9, 2>(), spread<18, 2>(),
                                 spread<6, 3>(), spread<9, 3>(), spread<18, 3>()};

// Below this an iteration on one compute unit takes no longer than the
// exchange.  20 iterations, one unit / spread: 3 x 6, p = 1000 61 / 87 us for
// 8 frames, p = 1600 95 / 87 for 1 and 96 / 100 for 16, p = 2000 114 / 89 and
// 115 / 109; 3 x 9, p = 1600 148 / 132 and 150 / 149, p = 2048 182 / 133 and
// 183 / 158.  Codes that no one-unit kernel takes (p = 1537 and more; the others
// have p < 64) are faster here at every length.
constexpr int kSpLeastP = 1800, kSpLeastLongP = 1024;

// Tries of a wavefront before it gives up, 1-2 us each.  LDPC_SPREAD_TRIES sets
// another number (read at each call); it changes speed, never results.
constexpr uint32_t kSpTries = 1u << 16;

uint32_t spread_tries() {
    const char* env = std::getenv("LDPC_SPREAD_TRIES");
    return env ? (uint32_t)std::strtoul(env, nullptr, 10) : kSpTries;
}

struct SpreadChoice {
    const SpreadVariant* v;
    int members, tb;
    size_t ticket, verdict, total;   // bytes: the boxes come first
};

// Codes that the one-unit decoder keeps two sums per variable for (its order
// of additions is the one followed here) and codes that no one-unit kernel
// takes (in the packages' arithmetic, so that a frame's results do not depend on
// the batch); batches that leave kSpMembers compute units to a frame: with 25
// frames on 10 units each the exchange's traffic makes it slower (p = 2000 133
// us for 115).
bool choose_spread(const ldpc_graph* g, int rule, int gamma, SpreadChoice& c) {
    const QCDesc& D = g->qc;
    if (g->kind != LDPC_GRAPH_QC || D.J != kSpRows || gamma < 1) return false;
    const char* path = std::getenv("LDPC_BLOCK_PATH");
    if (path && (std::strcmp(path, "onchip") == 0 || std::strcmp(path, "packages") == 0)) return false;
    const bool unit = onchip_fits(g);
    if (unit ? !onchip_pairs(g) || D.p < kSpLeastP : D.p < kSpLeastLongP) return false;
    for (int j = 0; j < D.J; ++j)
        if (D.rstart[j + 1] - D.rstart[j] != D.L) return false;   // a zero block
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    if (gamma > cus / kSpMembers || 2 * cus <= 32 * (kSpMembers - 1)) return false;
    c.tb = ((D.p + kSpMembers - 1) / kSpMembers + 63) / 64 * 64;
    if (c.tb > kSpThreads) return false;
    c.members = (D.p + c.tb - 1) / c.tb;
    c.v = nullptr;
    for (const SpreadVariant& v : kSpread)
        if (v.dc == D.L && v.rule == rule + (unit ? 0 : 2)) c.v = &v;
    c.verdict = (size_t)gamma * 2 * D.E * sizeof(uint64_t);
    c.ticket = c.verdict + (size_t)gamma * 2 * kSpMembers * sizeof(uint64_t);
    c.total = c.ticket + ((size_t)(1 + gamma) * sizeof(uint32_t) + 15) / 16 * 16;
    return c.v != nullptr;
}

}  // namespace

size_t spread_bytes(const ldpc_graph* g, int gamma) {
    SpreadChoice c;
    return choose_spread(g, 0, gamma, c) ? c.total : 0;
}

bool spread_in_place(const ldpc_graph* g, int gamma, const float* llr, const float* post, const uint8_t* bits) {
    const size_t count = (size_t)gamma * g->n;
    const uintptr_t a = reinterpret_cast<uintptr_t>(llr), b = reinterpret_cast<uintptr_t>(post);
    const uintptr_t c = reinterpret_cast<uintptr_t>(bits);
    return (a < b + 4 * count && b < a + 4 * count) || (a < c + count && c < a + 4 * count);
}

int spread_decode(const ldpc_graph* g, const float* llr, int gamma, int max_iters, int early, float* post,
                  uint8_t* bits, int32_t* iters, uint8_t* converged, void* ws, size_t ws_bytes, hipStream_t st,
                  const float* nms_w) {
    SpreadChoice c;
    if (!choose_spread(g, nms_w ? 1 : 0, gamma, c) || c.total > ws_bytes) return 0;
    if (spread_in_place(g, gamma, llr, post, bits)) return 0;
    const QCDesc& D = g->qc;
    char* base = reinterpret_cast<char*>(ws);
    SpreadArgs A{};
    A.llr = llr;
    A.post = post;
    A.bits = bits;
    A.iters = iters;
    A.conv = converged;
    A.nms_w = nms_w;
    A.box = reinterpret_cast<uint64_t*>(base);
    A.verdict = reinterpret_cast<uint64_t*>(base + c.verdict);
    A.ticket = reinterpret_cast<uint32_t*>(base + c.ticket);
    A.left = A.ticket + 1;
    A.tries = spread_tries();
    A.n = D.n;
    A.p = D.p;
    A.gamma = gamma;
    A.max_iters = max_iters;
    A.members = c.members;
    A.nb = D.nb;
    for (int j = 0; j < kSpRows; ++j) {
        A.rb0[j] = D.rstart[j];
        for (int k = 0; k < D.L; ++k) {
            const int a = D.eshift[D.rstart[j] + k];
            const int a1 = D.eshift[D.rstart[(j + 1) % kSpRows] + k], a2 = D.eshift[D.rstart[(j + 2) % kSpRows] + k];
            A.sh4[j * kSpSlots + k] = 4u * (uint32_t)a;
            A.to1[j * kSpSlots + k] = 8u * (uint32_t)((a - a1 + D.p) % D.p);
            A.to2[j * kSpSlots + k] = 8u * (uint32_t)((a - a2 + D.p) % D.p);
        }
    }
    timing::Scope ts(23, st);
    const size_t words = c.total / 16;
    spread_clear_kernel<<<(unsigned)std::min<size_t>((words + 255) / 256, 2048), 256, 0, st>>>(
        reinterpret_cast<uint4*>(base), words);
    if (hipGetLastError() != hipSuccess) return -1;
    void* args[] = {&A};
    return hipLaunchKernel(early ? c.v->fn_early : c.v->fn, dim3((unsigned)(gamma * c.members)), dim3((unsigned)c.tb),
                           args, 0, st) == hipSuccess ? 1 : -1;
}

}  // namespace ldpc
