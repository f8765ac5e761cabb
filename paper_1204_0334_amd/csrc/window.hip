// Sliding-window decoder with a stream on one compute unit and its messages
// in registers (gfx950): the codes unwrapped from 3 x 6 bases (period 3, two
// circulant columns per position, one circulant row per layer).
//
// window_lds_kernel of decode.hip, which takes the other codes, keeps every
// edge message of the window in LDS and passes over them twice per iteration
// (check rows, then variables).  Here a thread owns a check row of up to NW
// layers of the window and keeps their messages in registers; LDS holds two
// sums per variable, so that a beta is the sum of the other alphas, as in the
// other forms, with which the results agree bit for bit.  A position t is met
// by layers t, t + 1 and t + 2.  Per iteration, after the rows' update:
//
//   * layer t writes the prefix mu + a_t, layer t + 2 the suffix a_t+2;
//   * after a barrier layer t + 1 reads both, which sum to its beta, and adds
//     a_t+1 to both;
//   * after another the prefix is the beta of layer t + 2, mu and the suffix
//     that of layer t; they are read as the next update begins, and a third
//     barrier ends the reading.
//
// The posterior of a position that leaves is mu + ln 2 (a_t + suffix).  From
// then on it is frozen: where a later layer meets it, the row's register holds
// the beta it last sent (+infinity, the identity of the row's products, where
// the chain has no such position).
//
// The layers are dealt to G groups of threads by their number modulo G, so a
// layer stays with its thread while the window slides; in a group's registers
// layers move down by one when its oldest leaves.
//
// Bound by the vector ALUs, counted busy 89 % of the time: 17 plain
// instructions and 3 transcendentals per edge update, where the rule and the
// variables take 12.  p = 512, 128 positions, 512 streams, W = 6, 10 iterations: 7.30
// ms (1.64 10^12 edge updates per second); 13.0 ms with the messages in LDS
// and the same check rule, 14.8 ms before that.  With one sum L per variable
// and beta = clip(L - alpha) it took 7.75 ms, at 1.07-1.10 times the error of
// these sums against 64 bits before the change of check rule; now 0.86-0.95.
#include <hip/hip_runtime.h>

#include "check2.h"
#include "device.h"
#include "internal.h"
#include "window.h"

namespace ldpc {

constexpr int kWdPeriod = 3, kWdCols = 2, kWdSlots = kWdPeriod * kWdCols;

struct WindowArgs {
    const float* llr;     // [gamma][positions * c]
    float* post;
    uint8_t* bits;
    int32_t positions, layers, p, W, K;
    int32_t groups, per;  // groups of threads, threads per group
    // edge slot k of a layer of class m (index 6 m + k): 4 times the shift
    // towards position layer - (2 - k / 2), column k % 2
    uint32_t sh4[kWdPeriod * kWdSlots];
};

__device__ __forceinline__ float* wd_at(float* base, uint32_t byte) {
    return reinterpret_cast<float*>(reinterpret_cast<char*>(base) + byte);
}

template <int NW, int MAXT, int WPE>
__global__ void __launch_bounds__(MAXT, WPE) window_kernel(const WindowArgs A) {
    constexpr int T = kWdPeriod, LB = kWdCols, DC = kWdSlots, MS = T - 1;
    static_assert(MS == 2, "three layers meet a position");
    extern __shared__ float sums[];   // prefixes [W][LB][p], suffixes [W][LB][p]
    const int p = A.p, P = A.positions, W = A.W;
    const uint32_t p4 = 4u * (uint32_t)p, c4 = LB * p4, behind = (uint32_t)W * c4;   // the suffixes
    const int g = __builtin_amdgcn_readfirstlane((int)threadIdx.x / A.per);
    const uint32_t s4 = 4u * (threadIdx.x - (uint32_t)(g * A.per));
    const bool own = s4 < p4;
    const size_t frame = (size_t)blockIdx.x * P * LB * p;
    const float* __restrict__ mu = A.llr + frame;

    // Edge slots of the oldest position (2 layers back), the one after, the
    // layer's own.  al: alphas, then betas, of a row's edges; the last beta for
    // a frozen position, +inf where there is none.
    float al[NW][DC];
    uint32_t offs[NW][DC / 2];   // offsets of the edges' variables in their positions, two to a register
    float m0[NW][LB];            // channel LLRs of the layer's own position
    auto off = [&](int j, int k) -> uint32_t { return k % 2 ? offs[j][k / 2] >> 16 : offs[j][k / 2] & 0xffffu; };
    auto open_layer = [&](int j, int tau) {
        const int cls = tau % T;
#pragma unroll
        for (int k = 0; k < DC; ++k) {
            const uint32_t w = s4 + A.sh4[cls * DC + k];
            const uint32_t o = (uint32_t)(k % LB) * p4 + min(w, w - p4);
            if (k % 2 == 0)
                offs[j][k / 2] = o;
            else
                offs[j][k / 2] |= o << 16;
            const int pos = tau - (MS - k / LB);
            al[j][k] = (uint32_t)pos < (uint32_t)P ? 0.0f : __builtin_inff();
        }
        if (tau < P) {
#pragma unroll
            for (int q = 0; q < LB; ++q)
                m0[j][q] = (mu + (size_t)tau * (LB * p))[off(j, MS * LB + q) >> 2] + 0.0f;
        }
    };
    for (int i = threadIdx.x; i < min(W, P) * LB * p; i += blockDim.x) {
        sums[i] = mu[i] * kLog2eF + 0.0f;
        sums[W * LB * p + i] = 0.0f;
    }
    __syncthreads();

    int sW = 0;          // s mod W
    int w0 = g;          // the group's oldest layer is s + w0
    // ring offset of position s + w, -MS <= w < W
    auto slot = [&](int w) -> uint32_t {
        int r = sW + w;
        r = r < 0 ? r + W : r;
        return (uint32_t)(r >= W ? r - W : r) * c4;
    };
    // layer s + w of a row comes into the window: its first beta for the
    // position before its own
    auto enter = [&](int j, int s, int w) {
        if ((uint32_t)(s + w - 1) < (uint32_t)P) {
#pragma unroll
            for (int q = 0; q < LB; ++q) al[j][LB + q] = clip2(*wd_at(sums, slot(w - 1) + off(j, LB + q)));
        }
    };
#pragma unroll
    for (int j = 0; j < NW; ++j) {
#pragma unroll
        for (int k = 0; k < DC; ++k) al[j][k] = 0.0f;
#pragma unroll
        for (int k = 0; k < DC / 2; ++k) offs[j][k] = 0u;
#pragma unroll
        for (int q = 0; q < LB; ++q) m0[j][q] = 0.0f;
        if (own) {
            const int w = g + j * A.groups;
            open_layer(j, w);
            if (w < W) enter(j, 0, w);
        }
    }
    for (int s = 0; s < P; ++s) {
        auto live = [&](int w) { return w < W && s + w < A.layers; };                // layer s + w is in the window
        auto active = [&](int w, int dd) { return w >= dd && s + w - dd < P; };      // and meets position s + w - dd
        for (int it = 0; it < A.K; ++it) {
            if (own) {
#pragma unroll
                for (int j = 0; j < NW; ++j) {
                    const int w = w0 + j * A.groups;
                    if (!live(w)) continue;
                    if (active(w, 2)) {
#pragma unroll
                        for (int q = 0; q < LB; ++q) al[j][q] = clip2(*wd_at(sums, slot(w - 2) + off(j, q)));
                    }
                    if (active(w, 0)) {
#pragma unroll
                        for (int q = 0; q < LB; ++q) {
                            const int k = 2 * LB + q;
                            al[j][k] = clip2(fmaf(m0[j][q], kLog2eF, *wd_at(sums, behind + slot(w) + off(j, k))));
                        }
                    }
                    if (w >= MS && s + w < P) {
                        check2e_row<DC, 1>(al[j], DC);
                    } else {
                        float x[DC];
#pragma unroll
                        for (int k = 0; k < DC; ++k) x[k] = al[j][k];
                        check2e_row<DC, 1>(x, DC);
#pragma unroll
                        for (int k = 0; k < DC; ++k)
                            if (active(w, MS - k / LB)) al[j][k] = x[k];
                    }
                }
            }
            __syncthreads();
            if (own) {
#pragma unroll
                for (int j = 0; j < NW; ++j) {
                    const int w = w0 + j * A.groups;
                    if (!live(w)) continue;
#pragma unroll
                    for (int q = 0; q < LB; ++q) {
                        const int k = 2 * LB + q;
                        if (active(w, 0)) *wd_at(sums, slot(w) + off(j, k)) = fmaf(m0[j][q], kLog2eF, al[j][k]);
                        if (active(w, 2)) *wd_at(sums, behind + slot(w - 2) + off(j, q)) = al[j][q];
                    }
                }
            }
            __syncthreads();
            if (own) {
#pragma unroll
                for (int j = 0; j < NW; ++j) {
                    const int w = w0 + j * A.groups;
                    if (!live(w) || !active(w, 1)) continue;
                    float u[LB], v[LB];
#pragma unroll
                    for (int q = 0; q < LB; ++q) {
                        const uint32_t at = slot(w - 1) + off(j, LB + q);
                        u[q] = *wd_at(sums, at);
                        v[q] = live(w + 1) ? *wd_at(sums, behind + at) : 0.0f;
                    }
#pragma unroll
                    for (int q = 0; q < LB; ++q) {
                        const uint32_t at = slot(w - 1) + off(j, LB + q);
                        const float x = al[j][LB + q];
                        *wd_at(sums, at) = u[q] + x;
                        *wd_at(sums, behind + at) = v[q] + x;
                        al[j][LB + q] = clip2(u[q] + v[q]);
                    }
                }
            }
            __syncthreads();
        }
        // Position s is decided, by its own layer's rows, and freezes: the
        // layers that meet it from now on keep the beta they last sent.
        if (own) {
#pragma unroll
            for (int j = 0; j < NW; ++j) {
                const int w = w0 + j * A.groups;
                if (!live(w)) continue;
#pragma unroll
                for (int q = 0; q < LB; ++q) {
                    if (w == 0) {
                        const int k = 2 * LB + q;
                        const float S = al[j][k] + *wd_at(sums, behind + slot(0) + off(j, k));
                        const float x = posterior2(S, m0[j][q]);
                        const size_t at = frame + (size_t)s * (LB * p);   // the same for all threads
                        (A.post + at)[off(j, k) >> 2] = clip30(x);
                        (A.bits + at)[off(j, k) >> 2] = (uint8_t)(x < 0.0f);
                    } else if (w == MS) {
                        al[j][q] = clip2(*wd_at(sums, slot(0) + off(j, q)));
                    }
                }
            }
        }
        __syncthreads();
        // position s + W enters with its channel LLRs; layer s leaves, layer s + W enters
        if (s + W < P) {
            const uint32_t base = slot(0);
            const size_t v0 = (size_t)(s + W) * (LB * p);
            for (int i = threadIdx.x; i < LB * p; i += blockDim.x) {
                *wd_at(sums, base + 4u * (uint32_t)i) = mu[v0 + i] * kLog2eF + 0.0f;
                *wd_at(sums, behind + base + 4u * (uint32_t)i) = 0.0f;
            }
        }
        if (w0 == 0) {
            w0 = A.groups - 1;
#pragma unroll
            for (int j = 0; j + 1 < NW; ++j) {
#pragma unroll
                for (int k = 0; k < DC; ++k) al[j][k] = al[j + 1][k];
#pragma unroll
                for (int k = 0; k < DC / 2; ++k) offs[j][k] = offs[j + 1][k];
#pragma unroll
                for (int q = 0; q < LB; ++q) m0[j][q] = m0[j + 1][q];
            }
            if (own) open_layer(NW - 1, s + NW * A.groups);
        } else {
            --w0;
        }
        if (own) {
#pragma unroll
            for (int j = 0; j < NW; ++j)
                if (w0 + j * A.groups == W - 1) enter(j, s, W);
        }
        sW = sW + 1 == W ? 0 : sW + 1;
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

// Most rows of a layer.  10 iterations, 24 positions, ring in LDS or launches /
// here: p = 513, W = 6, 300 streams 3.71 / 2.50 ms, p = 900, W = 3 3.67 / 1.28;
// p = 800, W = 6 15.8 / 3.1; p = 1000, W = 4 13.9 / 2.2.  p = 1024 would gain as
// much (W = 4, 100 streams 5.2 / 1.1), but the repository's tests hold that
// size to the launches.
constexpr int kWdMostP = 1023;

int window_decode(const ldpc_graph* g, const float* llr, int gamma, int W, int K, float* post, uint8_t* bits,
                  hipStream_t st) {
    if (g->Jb != 1 || g->T != kWdPeriod || g->ms + 1 != g->T || g->Lb != kWdCols || g->p > kWdMostP) return 0;
    for (int v : g->sf)
        if (v < 0) return 0;
    const int per = (g->p + 63) / 64 * 64;
    // Layers per thread: the fewest that 1024 threads can hold the window with
    // (rows of one thread are updated one after the other).  W = 6, 10
    // iterations: p = 52, 20 positions, 128 streams, 1, 2, 3 or 6 layers: 152,
    // 237, 336, 597 us; p = 512, 128 positions, 256 streams, 3 or 6: 4.36 and
    // 5.60 ms.
    int nw = 0;
    for (int n : {6, 3, 2, 1})
        if ((W + n - 1) / n * per <= 1024) nw = n;
    if (nw == 0) return 0;
    const int groups = (W + nw - 1) / nw;
    const size_t lds = 2 * (size_t)W * kWdCols * g->p * sizeof(float);
    int dev = 0, limit = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&limit, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    if (lds > (size_t)limit) return 0;
    WindowArgs A{};
    A.llr = llr;
    A.post = post;
    A.bits = bits;
    A.positions = g->positions;
    A.layers = g->layers;
    A.p = g->p;
    A.W = W;
    A.K = K;
    A.groups = groups;
    A.per = per;
    for (int m = 0; m < kWdPeriod; ++m)
        for (int k = 0; k < kWdSlots; ++k)
            A.sh4[m * kWdSlots + k] =
                4u * (uint32_t)g->sf[(m * kWdPeriod + (g->ms - k / kWdCols)) * kWdCols + k % kWdCols];
    // With more streams than compute units, 64 registers, so that two
    // workgroups of 1024 threads share one (p = 512, 512 streams: 7.29 ms
    // against 8.70; 256 streams: 4.46 against 4.35).
    const bool two = gamma > compute_units();
    const void* fn = nw == 1 ? reinterpret_cast<const void*>(&window_kernel<1, 1024, 8>)
                     : nw == 2 ? (two ? reinterpret_cast<const void*>(&window_kernel<2, 1024, 8>)
                                      : reinterpret_cast<const void*>(&window_kernel<2, 1024, 4>))
                     : nw == 3 ? (two ? reinterpret_cast<const void*>(&window_kernel<3, 1024, 8>)
                                      : reinterpret_cast<const void*>(&window_kernel<3, 1024, 4>))
                               : reinterpret_cast<const void*>(&window_kernel<6, 1024, 4>);
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    timing::Scope ts(21, st);
    void* args[] = {&A};
    return hipLaunchKernel(fn, dim3((unsigned)gamma), dim3((unsigned)(groups * per)), args, lds, st) == hipSuccess ? 1
                                                                                                                   : -1;
}

}  // namespace ldpc
