// RGCN forward of a small graph in one launch, fp32, widths 32 and 64:
//   out[v] = act( sum over v's (relation r, destination v) runs of (1/c sum of X[src]) W[r]  +  X[v] W0 )
//
// On 10k edges the two kernels of the general plan (message rows per pair, weighted sum per destination) do microseconds of work
// between launches and dependent loads: 12.2 us.  Here a workgroup owns a destination: its eight half wavefronts take the runs in
// turn, each sums the run's input rows first and multiplies once, with the weight straight from L2, and the self-loop is one more
// run.  The chain is destination -> runs -> edges -> rows -> out, and nothing else waits.  The price is a weight per run
// instead of one per tile of pairs: sched_rgcn_small says up to where.
#include "rgnn_internal.h"
#include "traversal.h"
#include "device_utils.h"

#include <float.h>

namespace rgnn {

namespace {

struct SmallArgs {
    const int32_t* dst_run_ptr;
    const int32_t* run_ptr;
    const int32_t* run_rel;
    const int32_t* in_src;
    const float* X;
    const float* W;
    const float* W0;         // optional
    float* out;
    int norm, relu;
};

// (64 x 64 is given the registers of four wavefronts per SIMD: with fewer its rows of weights are not asked for together, 45 us
// instead of 41 with 128 runs per destination, 133 instead of 89 with 256)
template <int K, int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(K * D == 4096 ? 4 : 1, K * D == 4096 ? 4 : 8))) void rgcn_small_fwd_kernel(SmallArgs a) {
    constexpr int KR = K / 32, DR = D / 32;      // columns of a row per lane: lane + 32 * i
    __shared__ float red[8][D];
    const int v = blockIdx.x, lane = threadIdx.x & 31, half = threadIdx.x >> 5;
    const int q0 = a.dst_run_ptr[v], q1 = a.dst_run_ptr[v + 1], end = q1 + (a.W0 ? 1 : 0);
    float acc[DR];
#pragma unroll
    for (int n = 0; n < DR; ++n) acc[n] = 0.f;
    for (int q = q0 + half; q < end; q += 8) {
        const bool loop = q == q1;               // the self-loop: one row, weight W0
        const int qq = loop ? max(q1 - 1, 0) : q;
        const float* w = a.W0;
        float x[KR], f = 1.f;                    // f: what the run's product is multiplied by
        if (loop) {
#pragma unroll
            for (int k = 0; k < KR; ++k) x[k] = a.X[(size_t)v * K + lane + 32 * k];
        } else {
            const int b = a.run_ptr[qq], e = a.run_ptr[qq + 1];
            w = a.W + (size_t)a.run_rel[qq] * K * D;
#pragma unroll
            for (int k = 0; k < KR; ++k) x[k] = 0.f;
            for (int j0 = b; j0 < e; j0 += 32) {         // 32 sources per load, eight rows in flight
                const int src = a.in_src[min(j0 + lane, e - 1)], n = min(e - j0, 32);
                for (int j = 0; j < n; j += 8) {
                    float r[8][KR];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const size_t s = (size_t)__shfl(src, j + u, 32) * K + lane;
#pragma unroll
                        for (int k = 0; k < KR; ++k) r[u][k] = a.X[s + 32 * k];
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u)
#pragma unroll
                        for (int k = 0; k < KR; ++k) x[k] += j + u < n ? r[u][k] : 0.f;
                }
            }
            f = a.norm ? 1.f / (float)(e - b) : 1.f;
        }
        // a run's product is summed in four chains before it joins the sum over the runs (in one chain for all of them the error
        // of out at 64 x 64 and 100 relations was 2.0e-7 against 64 bits, the general plan's 1.5e-7; so: 1.0e-7)
        float t[4][DR];
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int n = 0; n < DR; ++n) t[p][n] = 0.f;
#pragma unroll
        for (int kr = 0; kr < KR; ++kr)
#pragma unroll
            for (int k = 0; k < 32; ++k) {
                const float xk = __shfl(x[kr], k, 32);
#pragma unroll
                for (int n = 0; n < DR; ++n) t[k & 3][n] += xk * w[(kr * 32 + k) * D + n * 32 + lane];
            }
#pragma unroll
        for (int n = 0; n < DR; ++n) acc[n] += f * ((t[0][n] + t[1][n]) + (t[2][n] + t[3][n]));
    }
    // The sum of a run's rows, or its product, may leave the range of fp32 where their mean does not: the columns that came out
    // infinite or NaN once more, from rows times a power of two that keeps the sum inside.  (Rows scaled from the start would
    // lose their last bits below 2^-118.)
    bool outside[DR], any = false;
#pragma unroll
    for (int n = 0; n < DR; ++n) any |= outside[n] = !(fabsf(acc[n]) <= FLT_MAX);
    if ((unsigned)(__ballot(any) >> (threadIdx.x & 32)) != 0) {       // in this half wavefront
        float again[DR];
#pragma unroll
        for (int n = 0; n < DR; ++n) again[n] = 0.f;
#pragma unroll 1
        for (int q = q0 + half; q < end; q += 8) {
            const bool loop = q == q1;
            const int b = loop ? v : a.run_ptr[q], e = loop ? v + 1 : a.run_ptr[q + 1];
            const float* const w = loop ? a.W0 : a.W + (size_t)a.run_rel[q] * K * D;
            const float share = pow2_share(e - b), f = (a.norm && !loop ? 1.f / (float)(e - b) : 1.f) / share;
            float x[KR], t[DR];
#pragma unroll
            for (int k = 0; k < KR; ++k) x[k] = 0.f;
#pragma unroll 1
            for (int j = b; j < e; ++j)
#pragma unroll
                for (int k = 0; k < KR; ++k) x[k] += share * a.X[(size_t)(loop ? v : a.in_src[j]) * K + lane + 32 * k];
#pragma unroll
            for (int n = 0; n < DR; ++n) t[n] = 0.f;
#pragma unroll
            for (int kr = 0; kr < KR; ++kr)
#pragma unroll 1
                for (int k = 0; k < 32; ++k) {
                    const float xk = __shfl(x[kr], k, 32);
#pragma unroll
                    for (int n = 0; n < DR; ++n) t[n] += xk * w[(kr * 32 + k) * D + n * 32 + lane];
                }
#pragma unroll
            for (int n = 0; n < DR; ++n) again[n] += f * t[n];
        }
#pragma unroll
        for (int n = 0; n < DR; ++n) acc[n] = outside[n] ? again[n] : acc[n];
    }
#pragma unroll
    for (int n = 0; n < DR; ++n) red[half][n * 32 + lane] = acc[n];
    __syncthreads();
    if (threadIdx.x < D) {
        float t = 0.f;
#pragma unroll
        for (int h = 0; h < 8; ++h) t += red[h][threadIdx.x];
        if (a.relu) t = t > 0.f ? t : 0.f;
        a.out[(size_t)v * D + threadIdx.x] = t;
    }
}

}  // namespace

rgnn_status_t rgcn_small_fwd(const rgnn_graph* g, int K, int D, const float* X, const float* W, const float* W0, int norm, int relu, float* out,
                             hipStream_t st) {
    if (g->N == 0) return RGNN_OK;
    const SmallArgs a{g->idx[RGNN_IDX_DST_RUN_PTR], g->idx[RGNN_IDX_RUN_PTR], g->idx[RGNN_IDX_RUN_REL], g->idx[RGNN_IDX_IN_SRC], X, W, W0, out, norm, relu};
    KernelTimer kt(st, "rgcn_small_fwd");
#define RGNN_SMALL(K_, D_) hipLaunchKernelGGL((rgcn_small_fwd_kernel<K_, D_>), dim3((unsigned)g->N), dim3(256), 0, st, a)
    if (K == 32 && D == 32) RGNN_SMALL(32, 32);
    else if (K == 32 && D == 64) RGNN_SMALL(32, 64);
    else if (K == 64 && D == 32) RGNN_SMALL(64, 32);
    else if (K == 64 && D == 64) RGNN_SMALL(64, 64);
    else RGNN_FAIL(RGNN_EUNSUPPORTED, "rgcn_small_fwd: widths %d -> %d not built", K, D);
#undef RGNN_SMALL
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

}  // namespace rgnn
