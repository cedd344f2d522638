// RGAT with one head, rows per (destination, relation) run: the backward's walks (the forward's are in rgat_fused.hip).
//
// With the inputs of a run summed before the product, out[v] = sum over v's runs q of w_q (A_q W[r]), A_q the sum of X[src_e] weighted within
// the run and w_q the run's weight in v.  Backward, dH_q = dOut[dst_q] W[r]^T is formed once per run (typed linear), and an edge
// e: u -> v of run q has
//   z_e = X[u] . wsp[r] + s_dst[q]  (wsp = W w_s),  att_e = exp(leakyrelu(z_e) - m_v) / s_v,  g_e = dOut[v] . (X[u] W[r]) = dH_q . X[u],
//   dz_e = att_e (g_e - dOut[v] . out[v]) (z_e > 0 ? 1 : slope),
// and adds att_e dH_q + dz_e wsp[r] to dX[u]: one walk over the edges of each source, which holds X[u] in registers and gathers the row dH_q,
// takes the place of the destination-major walk over the message rows, the pair-major sum and the sum of the pairs' input gradients.
#include "rgnn_internal.h"
#include "traversal.h"
#include "device_utils.h"
#include "schedule.h"

namespace rgnn {

namespace {

constexpr int kWalkThreads = 512;

// s_dst[q] = X[dst_q] . wtp[r_q], a group of D / 4 lanes per destination, whose row it reads once; wtp in LDS where it fits.
template <int D, bool LDSW>
__global__ __launch_bounds__(kWalkThreads) void rgat_run_logit_kernel(Items it, int R, const int32_t* __restrict__ run_rel,
                                                                      const float* __restrict__ X, const float* __restrict__ wtp, float* __restrict__ s_dst) {
    constexpr int LPR = D / 4, GPB = kWalkThreads / LPR;
    extern __shared__ __align__(16) float wtp_lds[];
    if (LDSW) {
        for (int i = threadIdx.x; i < R * D / 4; i += kWalkThreads) reinterpret_cast<float4*>(wtp_lds)[i] = reinterpret_cast<const float4*>(wtp)[i];
        __syncthreads();
    }
    // The next item's first relations and its row are asked for before this one's sums, and the ends of the one after it.  The items lie
    // by length, so that those of a wavefront end together.  900k destinations of width 64, us: one after the other 135; asked for ahead 122;
    // four sums at once 116; by length 102.
    const int c = threadIdx.x % LPR, step = gridDim.x * GPB, last = it.n - 1;
    int i = blockIdx.x * GPB + threadIdx.x / LPR;
    if (i >= it.n) return;
    int b = it.beg[i], e = it.end[i];
    int k1 = min(i + step, last), bn = it.beg[k1], en = it.end[k1], vn = it.row[k1];
    const int own = entry_of(c);                           // lane c's run of a chunk
    int rel = run_rel[max(min(b + own, e - 1), 0)];
    float4 x = *reinterpret_cast<const float4*>(X + (size_t)it.row[i] * D + c * 4);
    for (; i < it.n; i += step) {
        const int reln = run_rel[max(min(bn + own, en - 1), 0)];
        const float4 xn = *reinterpret_cast<const float4*>(X + (size_t)vn * D + c * 4);
        k1 = min(i + 2 * step, last);
        const int bnn = it.beg[k1], enn = it.end[k1], vnn = it.row[k1];
        for (int jc = b; jc < e; jc += LPR) {
            if (jc > b) rel = run_rel[min(jc + own, e - 1)];
            const int n = min(LPR, e - jc);
            float mine = 0.f;
#pragma unroll
            for (int k = 0; k < LPR; k += 4) {
                if (k >= n) break;
                float p[4];
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    p[t] = dot4(x, *reinterpret_cast<const float4*>((LDSW ? wtp_lds : wtp) + (size_t)group_lane<LPR>(rel, entry_of(k + t)) * D + c * 4));
                const float s = group_sum4<LPR>(p, c);
                mine = c >> 2 == k >> 2 ? s : mine;
            }
            if (own < n) s_dst[jc + own] = mine;
        }
        b = bn; e = en; bn = bnn; en = enn; rel = reln; x = xn; vn = vnn;
    }
}

// lq[q] = (leakyrelu(X[src] . wsp[r] + s_dst[q]), 1) of the runs with one edge; four runs at a time.
template <int D>
__global__ __launch_bounds__(256) void rgat_single_logits_kernel(int Q, const int32_t* __restrict__ run_ptr, const int32_t* __restrict__ run_rel,
                                                                 const int32_t* __restrict__ in_src, const float* __restrict__ X,
                                                                 const float* __restrict__ wsp, const float* __restrict__ s_dst, float slope,
                                                                 float2* __restrict__ lq) {
    constexpr int LPR = D / 4;
    const int64_t q0 = ((int64_t)blockIdx.x * (256 / LPR) + threadIdx.x / LPR) * 4;
    const int c = threadIdx.x % LPR;
    if (q0 >= Q) return;
    float p[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t q = min(q0 + u, (int64_t)Q - 1);
        p[u] = dot4(*reinterpret_cast<const float4*>(X + (size_t)in_src[run_ptr[q]] * D + c * 4),
                    *reinterpret_cast<const float4*>(wsp + (size_t)run_rel[q] * D + c * 4));
    }
    const float s = group_sum4<LPR>(p, c);
    const int64_t q = q0 + c;                              // lane c < 4 has run c's
    if (c < 4 && q < Q && run_ptr[q + 1] - run_ptr[q] == 1) {
        const float z = s + s_dst[q];
        lq[q] = make_float2(z > 0.f ? z : slope * z, 1.f);
    }
}

// A run's weight in its destination, for the weight gradient.  A lane per run.
__global__ __launch_bounds__(256) void rgat_run_weights_kernel(int Q, const int32_t* __restrict__ run_dst, const float2* __restrict__ ms,
                                                               const float2* __restrict__ lq, float* __restrict__ weight) {
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= Q) return;
    const float2 l = lq[q], st = ms[run_dst[q]];
    weight[q] = __expf(l.x - st.x) * l.y * (1.f / st.y);
}

// What the walk below needs of an edge's run: of a run with one edge its logit and dz, which is ds_dst as well, of the others s_dst and gbar.
// gbar_v = dOut[v] . out[v] is taken as the sum over v's runs of rowdot = weight dH_q . A_q, which the typed linear left (with dOut . out the
// error of dw_s against 64 bits was 4.7e-7 at 1.5M edges; so 2.9e-7, with the rows per pair 3.0e-7).  An edge that is alone in its destination
// so gets dz = 0 exactly, as with rows per pair.  Eight lanes per destination.
__global__ __launch_bounds__(256) void rgat_run_stat_kernel(int N, float slope, const int32_t* __restrict__ dst_run_ptr, const int32_t* __restrict__ run_ptr,
                                                            const float* __restrict__ rowdot, const float* __restrict__ weight,
                                                            const float2* __restrict__ ms, const float2* __restrict__ lq,
                                                            const float* __restrict__ s_dst, float4* __restrict__ stat, float* __restrict__ ds_dst) {
    // (four destinations at a time, the loads of their first eight runs independent: one by one 125 us at 900k destinations and 4.4M runs, so 93)
    constexpr int L = 8, V = 4;
    const int64_t v0 = ((int64_t)blockIdx.x * (256 / L) + threadIdx.x / L) * V;
    const int c = threadIdx.x % L;
    if (v0 >= N) return;
    int b[V], e[V];
    float2 st[V], l[V];
    float dot[V], w[V], sd[V], gbar[V];
    bool one[V];
#pragma unroll
    for (int u = 0; u < V; ++u) {
        const int64_t v = min(v0 + u, (int64_t)N - 1);
        b[u] = dst_run_ptr[v];
        e[u] = v0 + u < N ? dst_run_ptr[v + 1] : b[u];
        st[u] = ms[v];
    }
#pragma unroll
    for (int u = 0; u < V; ++u) {
        const int q = max(min(b[u] + c, e[u] - 1), 0);
        dot[u] = rowdot[q]; w[u] = weight[q]; l[u] = lq[q]; sd[u] = s_dst[q];
        one[u] = run_ptr[q + 1] - run_ptr[q] == 1;
        gbar[u] = b[u] + c < e[u] ? dot[u] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < V; ++u) {
        for (int q = b[u] + c + L; q < e[u]; q += L) gbar[u] += rowdot[q];
        gbar[u] = group_sum<L>(gbar[u]);
        const float inv = 1.f / st[u].y;
        for (int q = b[u] + c; q < e[u]; q += L) {
            if (q >= b[u] + L) {
                dot[u] = rowdot[q]; w[u] = weight[q]; l[u] = lq[q]; sd[u] = s_dst[q];
                one[u] = run_ptr[q + 1] - run_ptr[q] == 1;
            }
            const float dz = (dot[u] - w[u] * gbar[u]) * (l[u].x > 0.f ? 1.f : slope);
            stat[q] = make_float4(one[u] ? l[u].x : sd[u], st[u].x, inv, one[u] ? dz : gbar[u]);
            if (one[u]) ds_dst[q] = dz;
        }
    }
}

// ds_src of the pairs with more edges than a lane sums, a workgroup each: sum of the pair's dz, which lie together.
__global__ __launch_bounds__(256) void rgat_long_pair_kernel(const int32_t* __restrict__ ids, const int32_t* __restrict__ out_ptr,
                                                             const int32_t* __restrict__ pair_spos, const float* __restrict__ dz, float* __restrict__ ds_src) {
    __shared__ float red[4];
    const int p = ids[blockIdx.x], n = out_ptr[p + 1] - out_ptr[p];
    const float* const z = dz + pair_spos[p];
    float t0 = 0.f, t1 = 0.f;
    for (int i = threadIdx.x; i < n; i += 512) {
        t0 += z[i];
        if (i + 256 < n) t1 += z[i + 256];
    }
    const float t = group_sum<64>(t0 + t1);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) ds_src[p] = (red[0] + red[1]) + (red[2] + red[3]);
}

// A[r] = sum over r's pairs of ds_src[p] X[src_p] (ds_src the sum of the pair's dz) and U[r] = sum over r's runs of ds_dst[q] X[dst_q], by
// relation and block of nodes (plan_blocks in work_lists.h): a workgroup per item, whose groups of D / 4 lanes take D / 4 entries at a
// time, a lane each for what an entry needs.  7.3M pairs and 4.4M runs of 200 relations, width 64, 3 GB of rows: 530 us relation by relation,
// which read the nodes' rows from memory again for each, with another 105 for ds_src; so 294 for both.
struct BlockSumArgs {
    Items a, u;
    const int32_t* pair_src; const int32_t* pair_spos; const int32_t* out_ptr; const float* dz; const float* ds_src;
    const int32_t* relrun_idx; const int32_t* relrun_dst; const float* ds_dst;
    const float* X;
    float* A; float* a_partial; float* U; float* u_partial;
};
template <int D>
__global__ __launch_bounds__(256) void rgat_block_sums_kernel(BlockSumArgs s) {
    constexpr int LPR = D / 4, G = 256 / LPR;
    __shared__ float4 red[256];
    const bool pairs = (int)blockIdx.x < s.a.n;
    const int i = pairs ? blockIdx.x : blockIdx.x - s.a.n;
    const Items& it = pairs ? s.a : s.u;
    const int row = it.row[i];
    if (row < 0) return;
    const int b = it.beg[i], e = it.end[i], slot = it.slot[i];
    const int g = threadIdx.x / LPR, c = threadIdx.x % LPR;
    float4 acc0 = make_float4(0.f, 0.f, 0.f, 0.f), acc1 = acc0;
    auto entry = [&](int j, int& node, float& v) {         // (past the end the last entry with coefficient zero)
        const int jj = min(j, e - 1);
        if (pairs) {
            node = s.pair_src[jj];
            const int at = s.pair_spos[jj], n = s.out_ptr[jj + 1] - s.out_ptr[jj];
            v = s.dz[at];
            if (n > kSerialMax) v = s.ds_src[jj];
            else
                for (int k = 1; k < n; ++k) v += s.dz[at + k];
        } else {
            node = s.relrun_dst[jj];
            v = s.ds_dst[s.relrun_idx[jj]];
        }
        if (j >= e) v = 0.f;
    };
    int node = 0;
    float v = 0.f;
    if (b + g * LPR < e) entry(b + g * LPR + c, node, v);
    for (int jc = b + g * LPR; jc < e; jc += 256) {
        const int n0 = node, n = min(LPR, e - jc);
        const float v0 = v;
        if (jc + 256 < e) entry(jc + 256 + c, node, v);
#pragma unroll
        for (int k = 0; k < LPR; k += 4) {
            if (k >= n) break;
            float4 x[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) x[t] = *reinterpret_cast<const float4*>(s.X + (size_t)group_lane<LPR>(n0, k + t) * D + c * 4);
#pragma unroll
            for (int t = 0; t < 4; ++t) fma4(t & 1 ? acc1 : acc0, group_lane<LPR>(v0, k + t), x[t]);
        }
    }
    fma4(acc0, 1.f, acc1);
    red[threadIdx.x] = acc0;
    __syncthreads();
#pragma unroll
    for (int h = G / 2; h > 0; h /= 2) {
        if (g < h) fma4(red[threadIdx.x], 1.f, red[threadIdx.x + h * LPR]);
        __syncthreads();
    }
    if (g == 0) {
        float* const to = slot < 0 ? (pairs ? s.A : s.U) + (size_t)row * D : (pairs ? s.a_partial : s.u_partial) + (size_t)slot * D;
        reinterpret_cast<float4*>(to)[c] = red[c];
    }
}

struct SourceArgs {
    Items it;                 // edges by source
    const int32_t* src_row;   // [E] by source: row of the edge's run, the run, the relation
    const int32_t* src_run;
    const int32_t* src_rel;
    const float* X;           // [N][D]
    const float* dH;          // [Q][D]
    const float* wsp;         // [R][D]
    const float4* stat;       // [Q]
    float slope;
    int R, acc;
    float* dz;                // [E] by source
    float* dX;                // [N][D], or NULL: dz alone
    float* partial;
};

// A group of D / 4 lanes takes an item.  The indices of D / 4 edges are fetched at a time, lane c taking those of edge c, one chunk ahead of
// the rows, and handed round; nothing is reduced over a source's edges but the row, so pieces of popular sources are independent.
// The products of four edges are added up at once (group_sum4), and what follows from an edge's is formed by the lane that keeps the edge's
// numbers: 206 -> 199 us at 200k sources of width 128 and 2M edges, whose rows stay cached; where they do not, 660 either way.
template <int D, bool LDSW>
__device__ __forceinline__ void source_item(const SourceArgs& a, const float* wsp_lds, int i, int c) {
    constexpr int LPR = D / 4;
    const int b = a.it.beg[i], e = a.it.end[i], slot = a.it.slot[i];
    const size_t u = (size_t)a.it.row[i];
    float4 acc0 = make_float4(0.f, 0.f, 0.f, 0.f), acc1 = acc0;
    if (b < e) {
        const int own = entry_of(c);                       // lane c's edge of a chunk
        int jj = min(b + own, e - 1);
        int crow = a.src_row[jj], crun = a.src_run[jj], crel = a.src_rel[jj];
        const float4 x = *reinterpret_cast<const float4*>(a.X + u * D + c * 4);
        float4 cst = a.stat[crun & 0x7FFFFFFF];
        for (int jc = b; jc < e; jc += LPR) {
            const bool more = jc + LPR < e;
            int nrow = crow, nrun = crun, nrel = crel;
            if (more) {
                jj = min(jc + LPR + own, e - 1);
                nrow = a.src_row[jj];
                nrun = a.src_run[jj];
                nrel = a.src_rel[jj];
            }
            const int cend = min(LPR, e - jc);
            float mine = 0.f;                              // dz of edge jc + own
#pragma unroll
            for (int k = 0; k < LPR; k += 4) {
                if (k >= cend) break;
                float4 h[4], w[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) h[t] = *reinterpret_cast<const float4*>(a.dH + (size_t)group_lane<LPR>(crow, entry_of(k + t)) * D + c * 4);
                float pz[4], pg[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    w[t] = *reinterpret_cast<const float4*>((LDSW ? wsp_lds : a.wsp) + (size_t)group_lane<LPR>(crel, entry_of(k + t)) * D + c * 4);
                    pz[t] = dot4(x, w[t]);
                }
                const float z = group_sum4<LPR>(pz, c) + cst.x;
#pragma unroll
                for (int t = 0; t < 4; ++t) pg[t] = dot4(x, h[t]);
                const float g = group_sum4<LPR>(pg, c);
                // the lanes of quad k / 4 have their edges' sums, and form what follows from them
                float l = z > 0.f ? z : a.slope * z;
                l = crun < 0 ? cst.x : l;                  // the only edge of its run: the forward's logit, and dz
                const float al = __expf(l - cst.y) * cst.z;
                const float dz = crun < 0 ? cst.w : al * (g - cst.w) * (l > 0.f ? 1.f : a.slope);
                mine = c >> 2 == k >> 2 ? dz : mine;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float at = group_lane<LPR>(al, entry_of(k + t)), dt = group_lane<LPR>(dz, entry_of(k + t));
                    if (k + t < cend) {                    // (past the end the last edge again)
                        fma4(t & 1 ? acc1 : acc0, at, h[t]);
                        fma4(t & 1 ? acc1 : acc0, dt, w[t]);
                    }
                }
            }
            if (own < cend) a.dz[jc + own] = mine;
            if (more) {
                cst = a.stat[nrun & 0x7FFFFFFF];
                crow = nrow;
                crun = nrun;
                crel = nrel;
            }
        }
    }
    fma4(acc0, 1.f, acc1);
    if (slot < 0) {
        if (!a.dX) return;
        float4* o = reinterpret_cast<float4*>(a.dX + u * D + c * 4);
        if (a.acc) fma4(acc0, 1.f, *o);
        *o = acc0;
    } else {
        *reinterpret_cast<float4*>(a.partial + (size_t)slot * D + c * 4) = acc0;
    }
}

template <int D, bool LDSW>
__global__ __launch_bounds__(kWalkThreads) __attribute__((amdgpu_waves_per_eu(D == 128 ? 4 : 6))) void rgat_source_walk_kernel(SourceArgs a) {
    constexpr int LPR = D / 4, GPB = kWalkThreads / LPR;
    extern __shared__ __align__(16) float wsp_lds[];
    if (LDSW) {
        for (int i = threadIdx.x; i < a.R * D / 4; i += kWalkThreads) reinterpret_cast<float4*>(wsp_lds)[i] = reinterpret_cast<const float4*>(a.wsp)[i];
        __syncthreads();
    }
    for (int i = blockIdx.x * GPB + threadIdx.x / LPR; i < a.it.n; i += gridDim.x * GPB) source_item<D, LDSW>(a, wsp_lds, i, threadIdx.x % LPR);
}

}  // namespace

// a persistent kernel with the R folded vectors in LDS: as many workgroups as stay resident, never more than `need`
template <typename K>
static rgnn_status_t persistent_grid(const rgnn_graph* g, K kernel, size_t lds, size_t need, unsigned* grid) {
    const void* fn = reinterpret_cast<const void*>(kernel);
    if (lds) RGNN_TRY(allow_dynamic_lds(fn, lds));
    int per_cu = 1;
    RGNN_TRY(resident_blocks_per_cu(fn, kWalkThreads, lds, &per_cu));
    *grid = (unsigned)std::max<size_t>(1, std::min<size_t>(need, (size_t)per_cu * std::max(g->num_cus, 1)));
    return RGNN_OK;
}

template <int D, bool LDSW>
static rgnn_status_t launch_run_logit(const rgnn_graph* g, const float* X, const float* wtp, float* s_dst, hipStream_t st) {
    const size_t lds = LDSW ? (size_t)g->R * D * sizeof(float) : 0;
    unsigned grid = 1;
    RGNN_TRY(persistent_grid(g, rgat_run_logit_kernel<D, LDSW>, lds, blocks_for((size_t)g->dstrun_items.num_items, kWalkThreads / (D / 4)), &grid));
    hipLaunchKernelGGL((rgat_run_logit_kernel<D, LDSW>), dim3(grid), dim3(kWalkThreads), lds, st, dev_items(g->dstrun_items), g->R, g->idx[RGNN_IDX_RUN_REL], X, wtp, s_dst);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}
rgnn_status_t rgat_run_logit(const rgnn_graph* g, int K, const float* X, const float* wtp, float* s_dst, hipStream_t st) {
    if (g->Q == 0) return RGNN_OK;
    KernelTimer kt(st, "run_logit");
    if (sched_ws_in_lds(g->R, K)) RGNN_DISPATCH_D(K, return (launch_run_logit<DD, true>(g, X, wtp, s_dst, st)));
    else RGNN_DISPATCH_D(K, return (launch_run_logit<DD, false>(g, X, wtp, s_dst, st)));
}

rgnn_status_t rgat_single_logits(const rgnn_graph* g, int K, const float* X, const float* wsp, const float* s_dst, float slope, float* lq, hipStream_t st) {
    if (g->Q == 0) return RGNN_OK;
    KernelTimer kt(st, "single_logits");
    RGNN_DISPATCH_D(K, hipLaunchKernelGGL(rgat_single_logits_kernel<DD>, dim3(blocks_for(((size_t)g->Q + 3) / 4 * (DD / 4), 256)), dim3(256), 0, st, (int)g->Q,
                                          g->idx[RGNN_IDX_RUN_PTR], g->idx[RGNN_IDX_RUN_REL], g->idx[RGNN_IDX_IN_SRC], X, wsp, s_dst, slope,
                                          reinterpret_cast<float2*>(lq)));
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

rgnn_status_t rgat_run_weights(const rgnn_graph* g, const float* ms, const float* lq, float* weight, hipStream_t st) {
    if (g->Q == 0) return RGNN_OK;
    KernelTimer kt(st, "run_weights");
    hipLaunchKernelGGL(rgat_run_weights_kernel, dim3(blocks_for((size_t)g->Q, 256)), dim3(256), 0, st, (int)g->Q, g->idx[RGNN_IDX_RUN_DST],
                       reinterpret_cast<const float2*>(ms), reinterpret_cast<const float2*>(lq), weight);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

rgnn_status_t rgat_run_stat(const rgnn_graph* g, float slope, const float* rowdot, const float* weight, const float* ms, const float* lq, const float* s_dst,
                            float* stat, float* ds_dst, hipStream_t st) {
    if (g->Q == 0) return RGNN_OK;
    KernelTimer kt(st, "run_stat");
    hipLaunchKernelGGL(rgat_run_stat_kernel, dim3(blocks_for((size_t)g->N, 4 * 32)), dim3(256), 0, st, (int)g->N, slope, g->idx[RGNN_IDX_DST_RUN_PTR],
                       g->idx[RGNN_IDX_RUN_PTR], rowdot, weight, reinterpret_cast<const float2*>(ms), reinterpret_cast<const float2*>(lq), s_dst,
                       reinterpret_cast<float4*>(stat), ds_dst);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

rgnn_status_t rgat_block_sums(const rgnn_graph* g, int K, const float* X, const float* dz, float* ds_src, const float* ds_dst, float* A, float* a_partial,
                              float* U, float* u_partial, hipStream_t st) {
    if (g->long_pairs.n > 0) {
        KernelTimer kt(st, "ds_src_sum");
        hipLaunchKernelGGL(rgat_long_pair_kernel, dim3(g->long_pairs.n), dim3(256), 0, st, g->long_pairs.ids, g->idx[RGNN_IDX_OUT_PTR], g->pair_spos, dz, ds_src);
        RGNN_CHECK_LAUNCH();
    }
    const BlockSumArgs s{dev_items(g->pair_blocks), dev_items(g->run_blocks), g->idx[RGNN_IDX_PAIR_SRC], g->pair_spos, g->idx[RGNN_IDX_OUT_PTR], dz, ds_src,
                         g->idx[RGNN_IDX_RELRUN_IDX], g->relrun_dst, ds_dst, X, A, a_partial, U, u_partial};
    if (s.a.n + s.u.n == 0) return RGNN_OK;
    KernelTimer kt(st, "block_sums");
    RGNN_DISPATCH_D(K, hipLaunchKernelGGL(rgat_block_sums_kernel<DD>, dim3(s.a.n + s.u.n), dim3(256), 0, st, s));
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

template <int D, bool LDSW>
static rgnn_status_t launch_source_walk(const rgnn_graph* g, const SourceArgs& a, hipStream_t st) {
    const size_t lds = LDSW ? (size_t)g->R * D * sizeof(float) : 0;
    unsigned grid = 1;
    RGNN_TRY(persistent_grid(g, rgat_source_walk_kernel<D, LDSW>, lds, blocks_for((size_t)a.it.n, kWalkThreads / (D / 4)), &grid));
    hipLaunchKernelGGL((rgat_source_walk_kernel<D, LDSW>), dim3(grid), dim3(kWalkThreads), lds, st, a);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

rgnn_status_t rgat_source_walk(const rgnn_graph* g, int K, const float* X, const float* dH, const float* wsp, const float* stat, float slope, float* dz,
                               float* dX, bool acc, float* partial, hipStream_t st) {
    const ItemList& L = g->src_items;
    if (L.num_items == 0) return RGNN_OK;
    const SourceArgs a{dev_items(L), g->src_row, g->src_run, g->src_rel, X, dH, wsp, reinterpret_cast<const float4*>(stat), slope, g->R, acc, dz, dX, partial};
    {
        KernelTimer kt(st, "source_walk");
        if (sched_ws_in_lds(g->R, K)) RGNN_DISPATCH_D(K, RGNN_TRY((launch_source_walk<DD, true>(g, a, st))));
        else RGNN_DISPATCH_D(K, RGNN_TRY((launch_source_walk<DD, false>(g, a, st))));
    }
    if (!dX) return RGNN_OK;
    return combine_partials(L, K, partial, dX, 0, "source_walk.combine", st, nullptr, 1, 1, 0, acc ? dX : nullptr);
}

}  // namespace rgnn
