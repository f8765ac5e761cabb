// Pipelined decoder of LDPC convolutional codes (Algorithm 2) with a stream
// on one compute unit at a time (gfx950).
//
// The launch-per-slot form of decode.hip keeps the messages of all streams in
// a ring in memory and passes over them twice per slot and processor.  Here
// one workgroup takes one stream and K processors through the whole chain (a
// sweep), and I processors are ceil(I / K) sweeps, one launch each.  At slot
// t processor i = 1..K updates check layer t - (i-1) T (Algorithm 2's lag of
// ms + 1 = T frames):
//
//   * thread s owns check row s of every layer.  The messages alpha that
//     processor i leaves for processor i + 1, T slots later, stay in the
//     thread's registers; those of the last processor go to memory for the
//     next sweep;
//   * LDS holds sums L: of the positions the first processor reads, of
//     the 2 T positions between two processors (T being formed, T complete),
//     and of the T positions the last one forms.  A variable-to-check message
//     is clip(L - alpha) from the previous processor's complete sum, and a
//     layer's new messages are added into the positions it meets.  A layer
//     meets each variable of a position's circulant column once, so nothing
//     in a slot conflicts, whatever K is;
//   * the finished position of the last processor leaves (as sums for the
//     next sweep, or as posteriors and decisions) and the next position of the
//     first one enters in the following slot, in a ring position of their own
//     (RX = 1: one barrier per slot), or between two barriers where the LDS
//     has no room for those (RX = 0).
//
// Per processor every layer reads exactly the previous processor's complete
// sums, so the result is that of I flooding iterations, as in the other form;
// the arithmetic and its order are the other form's too (check2e_row over the
// row's slots, sums L from mu in order of the layers, beta = clip(L - alpha),
// for a layer's oldest position L as it was before its alpha came), and the
// two agree bit for bit.  The last processor's sums leave mu out: posteriors are
// mu + ln 2 times the sum of the alphas, so that the rounding of L does not
// come in.  The error of whole decodes against 64 bits is 0.93-1.02 of that of
// separate sums of the other alphas, which this form had before the sweeps;
// with L - alpha for every edge and posteriors from L it was 1.05-1.09.
//
// A sweep moves 8 bytes per edge and 8 per variable, and mu for each of its
// processors, through memory for K iterations.  For 3 x 6 that is the bound:
// p = 512, 512 streams, K = 3, counted 1.87 GB in and 1.09 GB out per sweep in
// the middle, at 5.5 TB/s (a plain copy reaches 5.05), the vector ALUs busy
// 74 % of the time.  4 x 24, p = 422, 256 streams, K = 2: 1.20 and 0.87 GB at
// 4.0 TB/s, the ALUs busy 52 %: two wavefronts on a SIMD, whose rows' chains
// from sums to new messages nothing hides.  So light rows issue all
// processors' reads first, and memory is read a slot ahead.  3 x 6 code, p = 512, 128 positions, 512 streams, 20 processors:
// 3.52 ms, 14.6 ms with two launches per slot; 4 x 24 code, p = 422, 64
// positions, 256 streams: 5.19 ms, 26.4 ms.  Before reads were issued early
// and the exchange shared the slot's barrier: 4.18 and 5.63 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "check2.h"
#include "device.h"
#include "internal.h"
#include "sweep.h"

namespace ldpc {

constexpr int kSwEdges = 96;   // shifts of all classes: T * T * Lb

struct SweepArgs {
    const float* llr;      // [gamma][positions * c], the batch's first stream
    float* post;           // [gamma][positions * c]
    uint8_t* bits;
    float* alpha;          // [batch][layers][T * Lb][p]: messages between sweeps
    float* sums;           // [batch][positions * c]: posterior sums between sweeps
    int32_t positions, layers, p;
    int32_t first, last;   // whether this is the first, the last sweep
    // edge slot k of a layer of class m (index m * T * Lb + k): 4 times the
    // shift of the circulant towards position layer - (T - 1 - k / Lb),
    // column k % Lb
    uint32_t sh4[kSwEdges];
};

// The element of an LDS array, of an array in memory, at a byte offset.
__device__ __forceinline__ float* sw_at(float* base, uint32_t byte) {
    return reinterpret_cast<float*>(reinterpret_cast<char*>(base) + byte);
}
template <typename V>
using Global = __attribute__((address_space(1))) V*;
template <typename V>
__device__ __forceinline__ Global<V> sw_at(Global<V> base, uint32_t byte) {
    // opaque here, so that the access takes a scalar base and a 32-bit offset
    asm volatile("" : "+v"(byte));
    return (Global<V>)((Global<char>)base + byte);
}

// A pointer into memory the same for the whole workgroup, moved to scalar
// registers (the compiler would keep running per-thread addresses instead).
template <typename V>
__device__ __forceinline__ Global<V> sw_uniform(V* at) {
    const uint64_t a = reinterpret_cast<uint64_t>(at);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return (Global<V>)((uint64_t)hi << 32 | lo);
}

// T: period = memory + 1; LB: circulant columns per position; K: processors;
// NB: blocks of check2e_row; GIN: the first processor reads its sums from
// memory, not from LDS (positions too large for it).
template <int T, int LB, int K, int NB, bool GIN, int RX, int MAXT, int WPE>
__global__ void __launch_bounds__(MAXT, WPE) sweep_kernel(const SweepArgs A) {
    constexpr int DC = T * LB, MS = T - 1, RD = T + RX;
    constexpr bool kPack = DC > 9;   // heavy rows: registers are scarce
    // [stage][position of the ring][column][p]: stage 0 (absent with GIN) and
    // stage K hold RD positions, the others 2 T
    extern __shared__ float ring[];
    const int p = A.p, P = A.positions;
    const uint32_t p4 = 4u * (uint32_t)p, c4 = LB * p4;
    const uint32_t s4 = 4u * threadIdx.x;
    const bool own = s4 < p4;
    const size_t stream = blockIdx.x;
    const size_t frame = stream * (size_t)P * LB * p;
    float* mu = const_cast<float*>(A.llr) + frame;
    float* sums = A.sums + frame;
    float* alpha = A.alpha + stream * (size_t)A.layers * DC * p;
    const bool first = A.first != 0, last = A.last != 0;
    // sums a sweep starts from: the channel LLRs in base-2 units (+ 0: no sum
    // is ever -0), or those the previous sweep left
    auto incoming = [&](float v) { return first ? v * kLog2eF + 0.0f : v; };
    float* in = first ? mu : sums;

    // what the rows of a layer keep between processors, by layer mod T: alphas,
    // and for the oldest position, whose sum their alphas completed, betas
    float fifo[K > 1 ? K - 1 : 1][T][DC];
    float head[DC], headn[DC];              // the same of the first processor's layer, of its next one
    float next[LB];                         // its next position's sums, as they are in memory
#pragma unroll
    for (int i = 0; i < (K > 1 ? K - 1 : 1); ++i)
#pragma unroll
        for (int m = 0; m < T; ++m)
#pragma unroll
            for (int k = 0; k < DC; ++k) fifo[i][m][k] = 0.0f;
#pragma unroll
    for (int k = 0; k < DC; ++k) head[k] = headn[k] = 0.0f;
#pragma unroll
    for (int q = 0; q < LB; ++q) next[q] = 0.0f;
    auto load_next = [&](int pos) {
        if (GIN || pos >= P) return;
        const Global<float> nt = sw_uniform(in + (size_t)pos * (LB * p));
#pragma unroll
        for (int q = 0; q < LB; ++q) next[q] = *sw_at(nt + q * p, s4);
    };
    if (own) {
        if (!GIN) {
#pragma unroll
            for (int q = 0; q < LB; ++q) *sw_at(ring, q * p4 + s4) = incoming(*sw_at(sw_uniform(in), q * p4 + s4));
        }
        if (!first) {
#pragma unroll
            for (int k = 0; k < DC; ++k) head[k] = *sw_at(sw_uniform(alpha), k * p4 + s4);
        }
        if (RX) load_next(1);
    }
    __syncthreads();

    // LDS offset of the ring of stage i
    auto stage = [&](int i) -> uint32_t {
        const int before = i == 0 ? 0 : (GIN ? 0 : RD) + (i - 1) * 2 * T;
        return (uint32_t)before * c4;
    };

    // memory reads for the next slot, a slot ahead of their use
    auto load_head = [&](int t, float (&to)[DC]) {
        if (first || t >= A.layers) return;
        const Global<float> at = sw_uniform(alpha + (size_t)t * (DC * p));
#pragma unroll
        for (int k = 0; k < DC; ++k) to[k] = *sw_at(at + k * p, s4);
    };
    auto prefetch = [&](int t) {
        load_next(t + 1 + RX);
        if (!kPack) load_head(t + 1, headn);
    };
    // ring offset of position pos, known to be r mod T, at stage 0 or K
    auto end_of = [&](int st, int pos, int r) -> uint32_t {
        return stage(st) + (uint32_t)(RX ? (pos + RD) % RD : r) * c4;
    };

    // slot t = T u + M
    auto slot = [&](int u, auto residue, auto whole) {
        constexpr int M = decltype(residue)::value;
        constexpr bool FULL = decltype(whole)::value;   // every processor's layer meets T positions
        const int t = T * u + M;
        // Offset of each edge's variable within its position, the same for all
        // processors.  Rows of weight <= 9 hold those of all T classes for the
        // whole sweep (the compiler's choice); heavier ones work this slot's
        // out, two to a register.
        uint32_t offs[DC], s4o = s4;
        if (kPack) asm volatile("" : "+v"(s4o));
#pragma unroll
        for (int k = 0; k < DC; ++k) {
            const uint32_t w = s4o + A.sh4[M * DC + k];
            const uint32_t o = (uint32_t)(k % LB) * p4 + min(w, w - p4);
            if (!kPack)
                offs[k] = o;
            else if (k % 2 == 0)
                offs[k / 2] = o;
            else
                offs[k / 2] |= o << 16;
        }
        if constexpr (kPack) {
            static_assert(DC % 2 == 0 || !kPack, "two offsets to a register");
#pragma unroll
            for (int k = 0; k < DC / 2; ++k) asm volatile("" : "+v"(offs[k]));
        }
        auto off = [&](int k) -> uint32_t {
            return !kPack ? offs[k] : k % 2 == 0 ? offs[k / 2] & 0xffffu : offs[k / 2] >> 16;
        };
        const uint32_t half[2] = {(uint32_t)(u & 1) * T * c4, (uint32_t)(1 - (u & 1)) * T * c4};
        // ring offset of position layer - dd of processor i's layer, at stage st
        auto where = [&](int st, int i, int dd) -> uint32_t {
            const int r = (M - dd + T) % T;
            if (st == 0 || st == K) return end_of(st, t - T * (i - 1) - dd, r);
            return (uint32_t)r * c4 + stage(st) + half[((i - 1) + (dd > M ? 1 : 0)) & 1];
        };
        auto there = [&](int i, int dd) { return FULL || (uint32_t)(t - T * (i - 1) - dd) < (uint32_t)P; };
        auto busy = [&](int i) { return FULL || (uint32_t)(t - T * (i - 1)) < (uint32_t)A.layers; };
        // what processor i's row needs: the channel LLRs that the position it
        // meets first starts from, its inputs, and the partial sums its new
        // messages go to, read before any is written (the compiler cannot know
        // that they differ)
        auto load_mu = [&](int i, float (&m0)[LB]) {
            if (!there(i, 0)) return;
            const Global<float> mt = sw_uniform(mu + (size_t)(t - T * (i - 1)) * (LB * p));
#pragma unroll
            for (int q = 0; q < LB; ++q) m0[q] = *sw_at(mt, off(MS * LB + q));
        };
        auto inputs = [&](int i, float (&x)[DC]) {
#pragma unroll
            for (int dd = MS; dd >= 0; --dd) {
                if (there(i, dd)) {
                    auto held = [&](int k) { return i == 1 ? head[k] : fifo[i >= 2 ? i - 2 : 0][M][k]; };
                    if (dd == MS && (i > 1 || !first)) {
#pragma unroll
                        for (int q = 0; q < LB; ++q) x[q] = held(q);
                        continue;
                    }
                    float L[LB];
                    if (GIN && i == 1) {
                        const Global<float> lt = sw_uniform(in + (size_t)(t - dd) * (LB * p));
#pragma unroll
                        for (int q = 0; q < LB; ++q) L[q] = incoming(*sw_at(lt, off((MS - dd) * LB + q)));
                    } else {
                        const uint32_t base = where(i - 1, i, dd);
#pragma unroll
                        for (int q = 0; q < LB; ++q) L[q] = *sw_at(ring, base + off((MS - dd) * LB + q));
                    }
#pragma unroll
                    for (int q = 0; q < LB; ++q) {
                        const int k = (MS - dd) * LB + q;
                        x[k] = clip2(L[q] - held(k));
                    }
                } else {
                    // no such edge: the identity of the row's products
#pragma unroll
                    for (int q = 0; q < LB; ++q) x[(MS - dd) * LB + q] = __builtin_inff();
                }
            }
        };
        auto partial = [&](int i, int dd, float (&v)[DC]) {
            const uint32_t base = where(i, i, dd);
#pragma unroll
            for (int q = 0; q < LB; ++q) v[(MS - dd) * LB + q] = *sw_at(ring, base + off((MS - dd) * LB + q));
        };
        auto partials = [&](int i, float (&v)[DC]) {
#pragma unroll
            for (int dd = MS; dd >= 1; --dd)
                if (there(i, dd)) partial(i, dd, v);
        };
        // x, the new messages, become what the rows keep
        auto add = [&](int i, const float (&m0)[LB], float (&v)[DC], float (&x)[DC]) {
#pragma unroll
            for (int dd = MS; dd >= 0; --dd) {
                if (!there(i, dd)) continue;
                const uint32_t base = where(i, i, dd);
                if (kPack && dd > 0) partial(i, dd, v);
#pragma unroll
                for (int q = 0; q < LB; ++q) {
                    const int k = (MS - dd) * LB + q;
                    // the last processor's sums are those of the alphas alone
                    const float sum = dd > 0 ? v[k] + x[k]
                                      : i == K && last ? 0.0f + x[k] : fmaf(m0[q] + 0.0f, kLog2eF, x[k]);
                    *sw_at(ring, base + off(k)) = sum;
                    if (dd == MS) x[k] = clip2(v[k]);
                }
            }
        };
        auto hand_on = [&](int i, const float (&x)[DC]) {
            if (i < K) {
#pragma unroll
                for (int k = 0; k < DC; ++k) fifo[i - 1 < K - 1 ? i - 1 : 0][M][k] = x[k];
            } else if (!last) {
                const Global<float> at = sw_uniform(alpha + (size_t)(t - T * (K - 1)) * (DC * p));
#pragma unroll
                for (int k = 0; k < DC; ++k) *sw_at(at + k * p, s4) = x[k];
            }
        };
        if constexpr (FULL && !kPack) {
            // light rows: every processor's reads go out first
            float m0[K][LB], x[K][DC], v[K][DC];
#pragma unroll
            for (int i = K; i >= 1; --i) load_mu(i, m0[i - 1]);
            prefetch(t);
#pragma unroll
            for (int i = K; i >= 1; --i) {
                inputs(i, x[i - 1]);
                partials(i, v[i - 1]);
            }
#pragma unroll
            for (int i = K; i >= 1; --i) {
                check2e_row<DC, NB>(x[i - 1], DC);
                add(i, m0[i - 1], v[i - 1], x[i - 1]);
            }
#pragma unroll
            for (int i = K; i >= 1; --i) hand_on(i, x[i - 1]);
        } else {
            prefetch(t);
#pragma unroll
            for (int i = K; i >= 1; --i) {
                if (!busy(i)) continue;
                float m0[LB], x[DC], v[DC];
                load_mu(i, m0);
                inputs(i, x);
                if (!kPack) partials(i, v);
                check2e_row<DC, NB>(x, DC);
                add(i, m0, v, x);
                hand_on(i, x);
            }
        }
    };
    // the last processor's finished position leaves, the first one's next
    // position enters
    auto exchange = [&](int u, auto residue) {
        constexpr int M = decltype(residue)::value;
        const int t = T * u + M;
        const int f = t - RX - T * (K - 1) - MS;
        if (f >= 0 && f < P) {
            const uint32_t base = end_of(K, f, (M + 1) % T);
#pragma unroll
            for (int q = 0; q < LB; ++q) {
                const float L = *sw_at(ring, base + q * p4 + s4);
                const size_t v = (size_t)f * (LB * p) + (size_t)q * p;
                if (last) {
                    const float x = posterior2(L, *sw_at(sw_uniform(mu + v), s4));
                    *sw_at(sw_uniform(A.post + frame + v), s4) = clip30(x);
                    sw_uniform(A.bits + frame + v)[threadIdx.x] = (uint8_t)(x < 0.0f);
                } else {
                    *sw_at(sw_uniform(sums + v), s4) = L;
                }
            }
        }
        if (!GIN && t + 1 < P) {
            const uint32_t base = end_of(0, t + 1, (M + 1) % T);
#pragma unroll
            for (int q = 0; q < LB; ++q) *sw_at(ring, base + q * p4 + s4) = incoming(next[q]);
        }
    };
    auto step = [&](int u, auto residue) {
        constexpr int M = decltype(residue)::value;
        const int t = T * u + M;
        if (own) {
            if (RX) exchange(u, residue);
            if (t - T * (K - 1) >= MS && t < P)
                slot(u, residue, std::true_type{});
            else
                slot(u, residue, std::false_type{});
            if (kPack) {
                load_head(t + 1, head);
            } else {
#pragma unroll
                for (int k = 0; k < DC; ++k) head[k] = headn[k];
            }
        }
        __syncthreads();
        if (!RX) {
            if (own) exchange(u, residue);
            __syncthreads();
        }
    };
    const int slots = P + MS + T * (K - 1) + RX;
    for (int block = 0; T * block < slots; ++block) {
        const int u = __builtin_amdgcn_readfirstlane(block);
        step(u, std::integral_constant<int, 0>{});
        step(u, std::integral_constant<int, 1>{});
        step(u, std::integral_constant<int, 2>{});
        if constexpr (T == 4) step(u, std::integral_constant<int, 3>{});
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

namespace {

struct SweepVariant {
    int T, Lb, K, rx;
    bool gin;
    int maxt;
    const void* fn;
};

template <int T, int LB, int K, int NB, bool GIN, int RX, int MAXT, int WPE>
constexpr SweepVariant sweep() {
    return SweepVariant{T, LB, K, RX, GIN, MAXT,
                        reinterpret_cast<const void*>(&sweep_kernel<T, LB, K, NB, GIN, RX, MAXT, WPE>)};
}

const SweepVariant kSweeps[] = {
    sweep<3, 2, 1, 1, false, 1, 512, 2>(), sweep<3, 2, 2, 1, false, 1, 512, 2>(), sweep<3, 2, 3, 1, false, 1, 512, 4>(),
    sweep<3, 2, 4, 1, false, 1, 512, 2>(), sweep<3, 2, 5, 1, false, 1, 512, 2>(),
    sweep<4, 6, 1, 2, false, 1, 512, 2>(), sweep<4, 6, 2, 2, false, 0, 512, 2>(),
    sweep<4, 6, 1, 2, false, 1, 1024, 4>(), sweep<4, 6, 1, 2, true, 1, 1024, 4>(),
};

size_t ring_bytes(const SweepVariant& v, const ldpc_graph* g) {
    const size_t positions = (v.gin ? 1 : 2) * (size_t)(v.T + v.rx) + (size_t)(v.K - 1) * 2 * v.T;
    return positions * v.Lb * g->p * sizeof(float);
}

// The variant of K processors for g, or NULL.
const SweepVariant* variant_for(const ldpc_graph* g, int K, size_t limit) {
    for (const SweepVariant& v : kSweeps)
        if (v.T == g->T && v.Lb == g->Lb && v.K == K && g->p <= v.maxt && ring_bytes(v, g) <= limit) return &v;
    return nullptr;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Processors per sweep of a code that the LDS (its size in limit) holds, 0 when
// the sweeps do not cover it.
int most_processors(const ldpc_graph* g, size_t& limit) {
    if (g->kind != LDPC_GRAPH_CONV || g->Jb != 1 || g->ms + 1 != g->T) return 0;
    for (int v : g->sf)
        if (v < 0) return 0;
    int dev = 0, bytes = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&bytes, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) {
        (void)hipGetLastError();
        bytes = 160 * 1024;   // sizing without a device (gfx950's LDS)
    }
    limit = (size_t)bytes;
    int most = 0;
    for (const SweepVariant& v : kSweeps)
        if (variant_for(g, v.K, limit)) most = std::max(most, v.K);
    return most;
}

}  // namespace

bool sweep_takes(const ldpc_graph* g) {
    size_t limit = 0;
    return most_processors(g, limit) > 0;
}

bool sweep_plan(const ldpc_graph* g, int gamma, int iters, SweepPlan& plan) {
    int most = most_processors(g, plan.lds_limit);
    if (most == 0) return false;
    // With more streams than compute units, two workgroups of three processors
    // or more on one are better than one of five (3 x 6, p = 512, 512 streams,
    // 20 processors: 3.53 ms against 3.79; 256 streams, one to a unit: 2.50
    // against 1.90), two of fewer are not (4 x 24, p = 422: 6.12 ms for K = 1
    // against 4.59 for K = 2).
    const int cus = compute_units();
    if (gamma > cus) {
        int twice = 0;
        for (const SweepVariant& v : kSweeps)
            if (variant_for(g, v.K, plan.lds_limit / 2)) twice = std::max(twice, v.K);
        if (twice >= 3) most = twice;
    }
    plan.sweeps = (iters + most - 1) / most;
    const size_t c = (size_t)g->Lb * g->p;
    plan.alpha_floats = plan.sweeps > 1 ? (size_t)g->layers * g->T * c : 0;
    plan.sum_floats = plan.sweeps > 1 ? (size_t)g->positions * c : 0;
    const size_t per = (plan.alpha_floats + plan.sum_floats) * sizeof(float);
    const size_t fit = per ? kSweepMostBytes / per : (size_t)gamma;
    if (fit < (size_t)std::min(gamma, cus)) return false;
    const int batches = (int)(((size_t)gamma + fit - 1) / fit);
    plan.batch = (gamma + batches - 1) / batches;
    plan.bytes = align256((size_t)plan.batch * plan.alpha_floats * sizeof(float)) +
                 align256((size_t)plan.batch * plan.sum_floats * sizeof(float));
    return true;
}

bool sweep_decode(const ldpc_graph* g, const SweepPlan& plan, const float* llr, int gamma, int iters, float* post,
                  uint8_t* bits, void* workspace, hipStream_t st) {
    SweepArgs A{};
    A.positions = g->positions;
    A.layers = g->layers;
    A.p = g->p;
    A.alpha = reinterpret_cast<float*>(workspace);
    A.sums = reinterpret_cast<float*>(reinterpret_cast<char*>(workspace) +
                                      align256((size_t)plan.batch * plan.alpha_floats * sizeof(float)));
    const int dc = g->T * g->Lb;
    for (int m = 0; m < g->T; ++m)
        for (int k = 0; k < dc; ++k)
            A.sh4[m * dc + k] = 4u * (uint32_t)g->sf[(m * g->T + (g->ms - k / g->Lb)) * g->Lb + k % g->Lb];
    const size_t n = (size_t)g->positions * g->Lb * g->p;
    for (int f = 0; f < gamma; f += plan.batch) {
        const int streams = std::min(plan.batch, gamma - f);
        A.llr = llr + (size_t)f * n;
        A.post = post + (size_t)f * n;
        A.bits = bits + (size_t)f * n;
        for (int s = 0; s < plan.sweeps; ++s) {
            const int K = iters / plan.sweeps + (s < iters % plan.sweeps ? 1 : 0);
            const SweepVariant* v = variant_for(g, K, plan.lds_limit);
            if (!v) return false;
            const size_t lds = ring_bytes(*v, g);
            A.first = s == 0;
            A.last = s == plan.sweeps - 1;
            if (hipFuncSetAttribute(v->fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
                return false;
            timing::Scope ts(10, st);
            void* args[] = {&A};
            if (hipLaunchKernel(v->fn, dim3((unsigned)streams), dim3((unsigned)((g->p + 63) / 64 * 64)), args, lds,
                                st) != hipSuccess)
                return false;
        }
    }
    return true;
}

}  // namespace ldpc
