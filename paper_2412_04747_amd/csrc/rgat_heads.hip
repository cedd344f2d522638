// Pieces of multi-head RGAT that the single-head path does not have.  With H heads the d_out
// columns split into H slices of d_out / H; head h of an edge uses the slices of hs, ht, w_s[r]
// and w_t[r] (the single-head formulas of the thesis' RGAT listing, applied per slice, outputs
// concatenated).  The rest of the multi-head path reuses the typed-linear kernels, the per-head
// softmax / edge-dot kernels of the HGT layer and the gather-sum with one coefficient per head.
#include "rgnn_internal.h"
#include "traversal.h"
#include "device_utils.h"

namespace rgnn {

// wv[r][h][k] = sum_{n in head h} W[r][k][n] * w[r][n]   (linear operator reordering, per head; the H vectors
// of a relation are adjacent, so the walks that need all of them touch one short block)
__global__ void fold_weight_heads_kernel(const float* __restrict__ W, const float* __restrict__ w, int R, int kd, int nd,
                                         int H, float* __restrict__ wv) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;   // (r, h, k)
    if (i >= H * R * kd) return;
    const int dh = nd / H;
    const int r = i / (H * kd), h = i / kd % H, k = i % kd;
    const float* Wr = W + ((size_t)r * kd + k) * nd + h * dh;
    const float* wr = w + (size_t)r * nd + h * dh;
    float s = 0.f;
    for (int n = 0; n < dh; ++n) s += Wr[n] * wr[n];
    wv[i] = s;
}

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

// Per relation r, with U[h][r] = sum_q ds_dst[q][h] X[dst_q] and h(n) the head of column n:
//   dw_t[r][n] = sum_k U[h(n)][r][k] W[r][k][n];   dW[r][k][n] += U[h(n)][r][k] * w_t[r][n]
// and, where A[r][h] = sum_p ds_src[p][h] X[src_p] is given (otherwise the caller forms dw_s from the message rows),
//   dw_s[r][n] = sum_k A[r][h(n)][k] W[r][k][n]
// Workgroups (r, j < nd / 32) form 32 columns of the vectors each (the eight lanes of a column take the k index in turn and are
// added in order through LDS); workgroups (r, nd / 32 + j) update 1024 consecutive elements of dW[r] each, four per lane (a lane's
// four columns are one head's).  nd is a power of two, at least 32.  (One workgroup per relation, a column per lane over all k: 38 us for 101 relations of width 64, now 8; 85 us for 60 of
// width 128, now 7.)
__global__ __launch_bounds__(256) void rgat_heads_param_finish_kernel(int R, int kd, int nd, int H, const float* __restrict__ W,
                                                                      const float* __restrict__ w_t, const float* __restrict__ U,
                                                                      const float* __restrict__ A, float* __restrict__ dW,
                                                                      float* __restrict__ dw_s, float* __restrict__ dw_t) {
    __shared__ float red[2][256];
    const int r = blockIdx.x, tid = threadIdx.x, ln = 31 - __clz(nd), ld = ln - (31 - __clz(H));     // log2 of a head's width
    const float* Wr = W + (size_t)r * kd * nd;
    const int vec_blocks = nd / 32;
    if ((int)blockIdx.y < vec_blocks) {
        const int n = blockIdx.y * 32 + (tid & 31), ks = tid >> 5, h = n >> ld;
        const float* Ur = U + ((size_t)h * R + r) * kd;
        const float* Ar = A + ((size_t)r * H + h) * kd;
        float s = 0.f, t = 0.f;
#pragma unroll 8
        for (int k = ks; k < kd; k += 8) {
            const float w = Wr[k * nd + n];
            t += Ur[k] * w;
            if (A) s += Ar[k] * w;
        }
        red[0][tid] = s;
        red[1][tid] = t;
        __syncthreads();
        if (ks == 0) {
            for (int q = 1; q < 8; ++q) {
                s += red[0][q * 32 + tid];
                t += red[1][q * 32 + tid];
            }
            if (A) dw_s[(size_t)r * nd + n] = s;
            dw_t[(size_t)r * nd + n] = t;
        }
        return;
    }
    const int i = ((blockIdx.y - vec_blocks) * 256 + tid) * 4;
    if (i >= kd * nd) return;
    const int k = i >> ln, n = i & (nd - 1);
    const float u = U[((size_t)(n >> ld) * R + r) * kd + k];
    const float4 wt = *reinterpret_cast<const float4*>(w_t + (size_t)r * nd + n);
    float4* o = reinterpret_cast<float4*>(dW + (size_t)r * kd * nd + i);
    float4 v = *o;
    v.x += u * wt.x;
    v.y += u * wt.y;
    v.z += u * wt.z;
    v.w += u * wt.w;
    *o = v;
}

// ---------------------------------------------------------------------------------------- launchers

rgnn_status_t fold_weight_heads(int R, int kd, int nd, int H, const float* W, const float* w, float* wv, hipStream_t st) {
    KernelTimer kt(st, "fold_weight");
    hipLaunchKernelGGL(fold_weight_heads_kernel, dim3(blocks_for((size_t)H * R * kd, 256)), dim3(256), 0, st, W, w, R, kd,
                       nd, H, wv);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

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

rgnn_status_t rgat_heads_param_finish(int R, int kd, int nd, int H, const float* W, const float* w_t, const float* U,
                                      const float* A, float* dW, float* dw_s, float* dw_t, hipStream_t st) {
    KernelTimer kt(st, "rgat_param_finish");
    hipLaunchKernelGGL(rgat_heads_param_finish_kernel, dim3(R, nd / 32 + (kd * nd + 1023) / 1024), dim3(256), 0, st, R, kd, nd, H, W, w_t, U, A, dW, dw_s, dw_t);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

}  // namespace rgnn
