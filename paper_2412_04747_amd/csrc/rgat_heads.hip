// Pieces of multi-head RGAT that the single-head path does not have.  With H heads the d_out
// columns split into H slices of d_out / H; head h of an edge uses the slices of hs, ht, w_s[r]
// and w_t[r] (the single-head formulas of the thesis' RGAT listing, applied per slice, outputs
// concatenated).  The rest of the multi-head path reuses the typed-linear kernels, the per-head
// softmax / edge-dot kernels of the HGT layer and the gather-sum with one coefficient per head.
#include "rgnn_internal.h"
#include "traversal.h"
#include "device_utils.h"

namespace rgnn {

// s_dst[q][h] = X[run_dst[q]] . wtp[run_rel[q]][h]: the run's X row is read once, one full-width dot per head; a lane
// group takes RPG consecutive runs so that four row reads or more (and the heads' folded vectors) are in flight per lane, and
// a lane stores all heads of a run (a store per run and head: 66 us for 1.1M runs and four heads, now 52).
template <int D, int H>
__global__ __launch_bounds__(256) void run_logit_heads_kernel(int Q, const int32_t* __restrict__ run_dst,
                                                              const int32_t* __restrict__ run_rel,
                                                              const float* __restrict__ X, const float* __restrict__ wtp,
                                                              float* __restrict__ s_dst) {
    constexpr int LPR = D / 4, RPG = 4;
    struct __align__(4 * (H < 4 ? H : 4)) Out { float v[H]; };
    const int q0 = (blockIdx.x * (256 / LPR) + threadIdx.x / LPR) * RPG, c4 = threadIdx.x % LPR;
    if (q0 >= Q) return;
    float4 x[RPG];
    int r[RPG];
#pragma unroll
    for (int u = 0; u < RPG; ++u) {
        const int q = min(q0 + u, Q - 1);
        x[u] = *reinterpret_cast<const float4*>(X + (size_t)run_dst[q] * D + c4 * 4);
        r[u] = run_rel[q];
    }
    Out mine;
#pragma unroll
    for (int h = 0; h < H; ++h) {
        float4 w[RPG];
#pragma unroll
        for (int u = 0; u < RPG; ++u) w[u] = *reinterpret_cast<const float4*>(wtp + ((size_t)r[u] * H + h) * D + c4 * 4);
        mine.v[h] = 0.f;
#pragma unroll
        for (int u = 0; u < RPG; ++u) {
            const float t = group_sum<LPR>(dot4(x[u], w[u]));
            if (c4 == u) mine.v[h] = t;
        }
    }
    if (c4 < RPG && q0 + c4 < Q) *reinterpret_cast<Out*>(s_dst + (size_t)(q0 + c4) * H) = mine;
}

// ---------------------------------------------------------------------------------------- launchers

rgnn_status_t run_logit_heads(const rgnn_graph* g, int D, int H, const float* X, const float* wtp, float* s_dst,
                              hipStream_t st) {
    if (g->Q == 0) return RGNN_OK;
    KernelTimer kt(st, "run_logit");
#define RGNN_RUN_LOGIT(H_) RGNN_DISPATCH_D(D, hipLaunchKernelGGL((run_logit_heads_kernel<DD, H_>), dim3(blocks_for((size_t)((g->Q + 3) / 4) * (DD / 4), 256)), \
                                                              dim3(256), 0, st, (int)g->Q, g->idx[RGNN_IDX_RUN_DST], g->idx[RGNN_IDX_RUN_REL], X, wtp, s_dst))
    if (H == 2) RGNN_RUN_LOGIT(2);
    else if (H == 4) RGNN_RUN_LOGIT(4);
    else if (H == 8) RGNN_RUN_LOGIT(8);
    else RGNN_FAIL(RGNN_EUNSUPPORTED, "run_logit_heads: %d heads not built (2, 4, 8)", H);
#undef RGNN_RUN_LOGIT
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

}  // namespace rgnn
