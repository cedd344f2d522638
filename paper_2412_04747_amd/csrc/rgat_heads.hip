// RGAT, rows per pair: the destination halves of the logits, for one head and for several.  With H heads the d_out columns split into H
// slices of d_out / H; head h of an edge uses the slices of hs, ht, w_s[r] and w_t[r] (the single-head formulas of the thesis'
// RGAT listing, applied per slice, outputs concatenated).
#include "rgnn_internal.h"
#include "traversal.h"
#include "device_utils.h"
#include "schedule.h"

#include <algorithm>

namespace rgnn {

// s_dst[q][h] = X[run_dst[q]] . wtp[run_rel[q]][h]: the run's X row is read once, one full-width dot per head; a lane
// group takes RPG consecutive runs so that four row reads or more (and the heads' folded vectors) are in flight per lane, and
// a lane stores all heads of a run (a store per run and head: 66 us for 1.1M runs of 101 relations and four heads, 55 so; 33 with the four
// runs' sums formed at once and the folded vectors in LDS, LDSW, the workgroups persistent).
template <int D, int H, bool LDSW>
__global__ __launch_bounds__(LDSW ? 1024 : 256) void run_logit_kernel(int Q, int R, const int32_t* __restrict__ run_dst,
                                                                            const int32_t* __restrict__ run_rel, const float* __restrict__ X,
                                                                            const float* __restrict__ wtp, float* __restrict__ s_dst) {
    constexpr int LPR = D / 4, RPG = 4;
    struct __align__(4 * (H < 4 ? H : 4)) Out { float v[H]; };
    extern __shared__ __align__(16) float wtp_lds[];
    if (LDSW) {
        for (int i = threadIdx.x; i < R * H * LPR; i += blockDim.x) reinterpret_cast<float4*>(wtp_lds)[i] = reinterpret_cast<const float4*>(wtp)[i];
        __syncthreads();
    }
    const float* const wv = LDSW ? wtp_lds : wtp;
    const int c4 = threadIdx.x % LPR, groups = blockDim.x / LPR, n4 = (Q - 1) / RPG + 1;
    for (int g = blockIdx.x * groups + threadIdx.x / LPR; g < n4; g += LDSW ? gridDim.x * groups : n4) {
        const int q0 = g * RPG;
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
            float p[RPG];
#pragma unroll
            for (int u = 0; u < RPG; ++u) p[u] = dot4(x[u], *reinterpret_cast<const float4*>(wv + ((size_t)r[u] * H + h) * D + c4 * 4));
            mine.v[h] = group_sum4<LPR>(p, c4);           // lane u < 4: run u's
        }
        if (c4 < RPG && q0 + c4 < Q) *reinterpret_cast<Out*>(s_dst + (size_t)(q0 + c4) * H) = mine;
    }
}

// ---------------------------------------------------------------------------------------- launchers

template <int D, int H>
static rgnn_status_t launch_run_logit(const rgnn_graph* g, const float* X, const float* wtp, float* s_dst, hipStream_t st) {
    const size_t lds = (size_t)g->R * H * D * sizeof(float), quads = ((size_t)g->Q + 3) / 4;
    const int32_t *dst = g->idx[RGNN_IDX_RUN_DST], *rel = g->idx[RGNN_IDX_RUN_REL];
    if (sched_halves_in_lds(g->R, H, D, g->Q)) {
        const void* fn = reinterpret_cast<const void*>(run_logit_kernel<D, H, true>);
        RGNN_TRY(allow_dynamic_lds(fn, lds));
        int per_cu = 1;
        RGNN_TRY(resident_blocks_per_cu(fn, 1024, lds, &per_cu));
        const size_t grid = std::min(blocks_for(quads, 1024 / (D / 4)), (unsigned)(per_cu * std::max(g->num_cus, 1)));
        hipLaunchKernelGGL((run_logit_kernel<D, H, true>), dim3((unsigned)grid), dim3(1024), lds, st, (int)g->Q, g->R, dst, rel, X, wtp, s_dst);
    } else {
        hipLaunchKernelGGL((run_logit_kernel<D, H, false>), dim3(blocks_for(quads * (D / 4), 256)), dim3(256), 0, st, (int)g->Q, g->R, dst, rel, X, wtp,
                           s_dst);
    }
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

rgnn_status_t run_logit(const rgnn_graph* g, int D, int H, const float* X, const float* wtp, float* s_dst, hipStream_t st) {
    if (g->Q == 0) return RGNN_OK;
    KernelTimer kt(st, "run_logit");
#define RGNN_RUN_LOGIT(H_) RGNN_DISPATCH_D(D, return (launch_run_logit<DD, H_>(g, X, wtp, s_dst, st)))
    if (H == 1) RGNN_RUN_LOGIT(1);
    else if (H == 2) RGNN_RUN_LOGIT(2);
    else if (H == 4) RGNN_RUN_LOGIT(4);
    else if (H == 8) RGNN_RUN_LOGIT(8);
    else RGNN_FAIL(RGNN_EUNSUPPORTED, "run_logit: %d heads not built (1, 2, 4, 8)", H);
#undef RGNN_RUN_LOGIT
    return RGNN_OK;
}

}  // namespace rgnn
