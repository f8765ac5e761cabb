// Message-package decoder of a short code with a frame's packages in LDS
// (gfx950).
//
// Short codes that the register kernels do not take (rows of weight above 9
// with p < 64, irregular bases) were decoded by two launches per iteration, 3.6
// us each however little there is to do: 160 us for 20 iterations of 3 x 18, p
// = 36.  Here a workgroup decodes one frame: its E messages, n channel LLRs and
// n posteriors lie in LDS, a thread takes check rows and then variables in
// turn, two barriers per iteration.  The arithmetic and the order of every sum
// are those of the launch-per-phase kernels (sp_check, sp_variable), so the
// results are theirs bit for bit.
//
// Early stopping: the rows of iteration it are tested with the decisions of
// it - 1 (the posteriors' signs) before the variables are updated, and the
// frame ends with the posteriors that are still there.
//
// Bound by latency while frames are few (4 us per iteration of 3 x 18, p = 36: a
// row's 18 loads, its sweep and two barriers), then by the vector ALUs (6000
// frames, 20 iterations: 565 us for 937 in launches).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>

#include "device.h"
#include "internal.h"
#include "onchip.h"
#include "small.h"

namespace ldpc {

struct SmallArgs {
    const float* llr;    // [gamma][n]
    float* post;         // [gamma][n]
    uint8_t* bits;       // [gamma][n]
    int32_t* iters;      // [gamma] or NULL
    uint8_t* conv;       // [gamma] or NULL
    int32_t max_iters, early;
};

// (first package, shift or column) of the edge blocks, in LDS
struct SmallEdge {
    int32_t base, shift;
};

// floats of LDS: messages, LLRs, posteriors, then the edges by row and by
// column, the rows' and columns' first blocks, the flags
size_t small_lds(const QCDesc& D) {
    return ((size_t)D.E + 2 * (size_t)D.n) * sizeof(float) + 2 * (size_t)D.nb * sizeof(SmallEdge) +
           (size_t)(D.J + 1 + D.L + 1 + 2) * sizeof(int32_t);
}

template <int DC, int DV>
__global__ void __launch_bounds__(512) small_kernel(const QCDesc D, const SmallArgs A) {
    extern __shared__ float msg[];   // [E]
    float* mu = msg + D.E;           // [n]
    float* post = mu + D.n;          // [n]
    SmallEdge* rowe = reinterpret_cast<SmallEdge*>(post + D.n);   // block b: first variable, shift
    SmallEdge* cole = rowe + D.nb;                                // entry of cedge: first package, shift
    int32_t* rstart = reinterpret_cast<int32_t*>(cole + D.nb);    // [J + 1]
    int32_t* cstart = rstart + D.J + 1;                           // [L + 1]
    int32_t* flag = cstart + D.L + 1;                             // [2]: iterations' violated rows
    const int tid = threadIdx.x, TB = blockDim.x, p = D.p;
    const size_t f0 = (size_t)blockIdx.x * D.n;
    for (int b = tid; b < D.nb; b += TB) {
        rowe[b] = SmallEdge{(int)D.ecol[b] * p, D.eshift[b]};
        const int c = D.cedge[b];
        cole[b] = SmallEdge{c * p, D.eshift[c]};
    }
    for (int j = tid; j <= D.J; j += TB) rstart[j] = D.rstart[j];
    for (int l = tid; l <= D.L; l += TB) cstart[l] = D.cstart[l];
    for (int v = tid; v < D.n; v += TB) mu[v] = A.llr[f0 + v];
    if (tid < 2) flag[tid] = 0;
    __syncthreads();
    // iteration 1 takes the channel LLRs as messages
    for (int e = tid; e < D.E; e += TB) {
        const int b = e / p, s = e - b * p;
        int t = s + rowe[b].shift;
        if (t >= p) t -= p;
        msg[e] = mu[rowe[b].base + t];
    }
    __syncthreads();

    int dmin = D.dc_max;   // no row is lighter
    for (int j = 0; j < D.J; ++j) dmin = min(dmin, (int)D.rstart[j + 1] - (int)D.rstart[j]);

    int it = 1, stop = 0;
    for (;; ++it) {
        // check rows of iteration it; the syndrome of it - 1
        const bool fin = it > A.max_iters;
        const bool syn = it >= 2 && (A.early || fin);
        bool viol = false;
        for (int r = tid; r < D.m; r += TB) {
            const int j = r / p, s = r - j * p;
            const int b0 = rstart[j], d = rstart[j + 1] - b0;
            if (d == 0) continue;
            // slots beyond the row's weight read its last edge again: no load
            // waits for another
            if (syn) {
                bool par = false;
#pragma unroll
                for (int k = 0; k < DC; ++k) {
                    const SmallEdge e = rowe[b0 + min(k, d - 1)];
                    const uint32_t t = (uint32_t)(s + e.shift);
                    const float L = post[e.base + (int)min(t, t - (uint32_t)p)];
                    par ^= k < d && L < 0.0f;
                }
                viol = viol || par;
            }
            if (fin) continue;
            float in[DC][1], out[DC][1];
#pragma unroll
            for (int k = 0; k < DC; ++k) in[k][0] = msg[(b0 + min(k, d - 1)) * p + s];
            sp_check<DC, 1>(in, d, out);
#pragma unroll
            for (int k = 0; k < DC; ++k)
                if (k < dmin || k < d) msg[(b0 + k) * p + s] = out[k][0];
        }
        if (syn && viol) flag[it & 1] = 1;
        __syncthreads();
        if (syn && flag[it & 1] == 0) {
            stop = it - 1;
            break;
        }
        if (fin) break;
        if (tid == 0) flag[(it + 1) & 1] = 0;
        // variables
        for (int v = tid; v < D.n; v += TB) {
            const int l = v / p, t = v - l * p;
            const int c0 = cstart[l], d = cstart[l + 1] - c0;
            int at[DV];
            float a[DV][1], b[DV][1], L[1];
#pragma unroll
            for (int k = 0; k < DV; ++k) {
                const SmallEdge e = cole[min(c0 + min(k, max(d - 1, 0)), D.nb - 1)];
                const uint32_t s = (uint32_t)(t - e.shift);
                at[k] = e.base + (int)min(s, s + (uint32_t)p);
                a[k][0] = msg[at[k]];
            }
#pragma unroll
            for (int k = 0; k < DV; ++k) a[k][0] = k < d ? a[k][0] : 0.0f;
            const float m[1] = {mu[v]};
            sp_variable<DV, 1>(m, a, b, L);
            post[v] = L[0];
#pragma unroll
            for (int k = 0; k < DV; ++k)
                if (k < d) msg[at[k]] = b[k][0];
        }
        __syncthreads();
    }
    for (int v = tid; v < D.n; v += TB) {
        A.post[f0 + v] = clip30(post[v]);
        A.bits[f0 + v] = (uint8_t)(post[v] < 0.0f);
    }
    if (tid == 0) {
        if (A.iters) A.iters[blockIdx.x] = A.early && stop ? stop : A.max_iters;
        if (A.conv) A.conv[blockIdx.x] = stop ? 1 : 0;
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

namespace {

struct SmallVariant {
    int dc, dv;
    const void* fn;
};

template <int DC, int DV>
constexpr SmallVariant small() {
    return SmallVariant{DC, DV, reinterpret_cast<const void*>(&small_kernel<DC, DV>)};
}

// the row capacities of the launch-per-phase kernels: the rounding of a full
// row's last slot depends on whether the capacity exceeds its weight
const SmallVariant kSmall[] = {small<4, 4>(),  small<4, 16>(),  small<6, 4>(),  small<6, 16>(), small<8, 4>(),
                               small<8, 16>(), small<12, 4>(),  small<12, 16>(), small<16, 4>(), small<16, 16>(),
                               small<24, 4>(), small<24, 16>(), small<32, 4>(), small<32, 16>()};

// Codes that no register kernel takes with up to kSmallEdges edges, where two
// launches per iteration (7 us at least) cost more than a frame's work; with
// columns of weight above 4 (16 slots per variable) while every frame has a
// compute unit to itself.  20 iterations, launches / here: 3 x 18, p = 36 220
// / 81 us for 1 frame, 485 / 151 for 1500; 4 x 24, p = 60 251 / 97 and 742 /
// 322; irregular 12 x 24, p = 27, columns of weight up to 12, 268 / 125 for 1
// frame, but 717 / 751 for 1500; 6 x 12, p = 400 (20,000 edges) 238 / 394.
constexpr int kSmallEdges = 8192;

const SmallVariant* choose_small(const ldpc_graph* g, int gamma, size_t& lds) {
    if (!g || g->kind != LDPC_GRAPH_QC || g->qc.E == 0 || g->qc.E > kSmallEdges || onchip_fits(g)) return nullptr;
    if (g->qc.dv_max > 4 && gamma > compute_units()) return nullptr;
    const char* path = std::getenv("LDPC_BLOCK_PATH");
    if (path && std::strcmp(path, "packages") == 0) return nullptr;
    int dev = 0, limit = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&limit, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    lds = small_lds(g->qc);
    if (lds > (size_t)limit) return nullptr;
    for (const SmallVariant& v : kSmall)
        if (v.dc >= g->qc.dc_max && v.dv >= g->qc.dv_max) return &v;
    return nullptr;
}

}  // namespace

bool small_selected(const ldpc_graph* g, int gamma) {
    size_t lds = 0;
    return choose_small(g, gamma, lds) != nullptr;
}

int small_decode(const ldpc_graph* g, const float* llr, int gamma, int max_iters, int early, float* post,
                 uint8_t* bits, int32_t* iters, uint8_t* converged, hipStream_t st) {
    size_t lds = 0;
    const SmallVariant* v = choose_small(g, gamma, lds);
    if (!v) return 0;
    const QCDesc& D = g->qc;
    SmallArgs A{llr, post, bits, iters, converged, max_iters, early};
    if (hipFuncSetAttribute(v->fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    // a thread for each row; while every frame has a compute unit to itself, for
    // each second variable too
    const int work = gamma <= compute_units() ? std::max(D.m, D.n / 2) : D.m;
    const int tb = std::min(512, std::max(64, (work + 63) / 64 * 64));
    timing::Scope ts(23, st);
    void* args[] = {const_cast<QCDesc*>(&D), &A};
    return hipLaunchKernel(v->fn, dim3((unsigned)gamma), dim3((unsigned)tb), args, lds, st) == hipSuccess ? 1 : -1;
}

}  // namespace ldpc
