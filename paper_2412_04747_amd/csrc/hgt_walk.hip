// Edge walks of the HGT layer: per-head attention logit, edge softmax and weighted sum of the messages, and their
// backward (caption of the thesis figure "HGT and RGAT layer").
//
// A (source, relation) pair's key row Ka[p] and message row M[p] lie side by side in KM[p][2][D]: both are needed for
// every edge of the pair, in the forward and in the backward walk, so an edge costs one gather of 2 D columns.  Three
// walks make up the layer:
//   forward, per destination:  logit = Ka . Q[v], running-maximum softmax per head, Z[v] = sum att M;  kept for the
//                              backward pass: (max, sum) per (destination, head), nothing per edge
//   backward, per destination: att recomputed from the key row and (max, sum); dl = att (dZ . M - dZ . Z);
//                              dQ[v] = sum dl Ka;  (att, dl) stored side by side per edge and head
//   backward, per pair:        dKM[p] = (sum dl Q[dst], sum att dZ[dst])
// All three are bound by the gathered rows.  On 20M edges (5.4M pairs, 2M nodes), width 128 in bf16, 4 heads, they take
// 2.01 + 2.48 + 2.05 ms: 5.6, 5.3 and 5.8 TB/s of the bytes they cannot avoid.  With the logits, softmax, weighted sum, edge
// dot and the three gradient sums as walks of their own (six gathers of D columns per edge, and weights stored and
// re-read per edge between them) the same work took 7.95 ms.
//
// A row of D columns is read by D / V lanes with 16-byte loads (V = 4 fp32 or 8 bf16 columns); the LPH lanes of a
// head reduce by DPP.  Arithmetic is fp32.  Weights come from expf: __expf is off by 2e-6 at a logit 60 below the maximum, expf by
// a rounding (no difference in time on the graphs above and at 2M edges, 1 % of the layer at 300k edges in fp32).
#include "rgnn_internal.h"
#include "traversal.h"
#include "device_utils.h"
#include "schedule.h"

namespace rgnn {

namespace {

__device__ __forceinline__ void widen_raw(rgnn_v4u t, float (&v)[8]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[2 * q] = __uint_as_float(t[q] << 16);
        v[2 * q + 1] = __uint_as_float(t[q] & 0xFFFF0000u);
    }
}
__device__ __forceinline__ void widen_raw(rgnn_v4u t, float (&v)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = __uint_as_float(t[q]);
}
// the 16 bytes of a row that belong to this lane, kept as loaded until they are used
template <typename T>
__device__ __forceinline__ rgnn_v4u load_raw(const T* p) { return *reinterpret_cast<const rgnn_v4u*>(p); }

// acc += sum of c[u] * row u over a batch.  fp32 rows: the batch is summed in two chains of its own first, one rounding at
// acc's magnitude per batch; bf16 rows are rounded to 8 bits in the end, and one chain does.
template <typename T, int V, int NE>
__device__ __forceinline__ void add_rows(float (&acc)[V], const float (&c)[NE], const rgnn_v4u (&rows)[NE]) {
    float t0[V], t1[V];
    zero_cols(t0);
    zero_cols(t1);
#pragma unroll
    for (int u = 0; u < NE; ++u) {
        float v[V];
        widen_raw(rows[u], v);
        if (sizeof(T) == 2) fma_cols(acc, c[u], v);
        else if (2 * u < NE) fma_cols(t0, c[u], v);
        else fma_cols(t1, c[u], v);
    }
    if (sizeof(T) == 4) {
#pragma unroll
        for (int q = 0; q < V; ++q) acc[q] += t0[q] + t1[q];
    }
}

struct WalkArgs {
    Items it;
    int wide_n, wide_blocks;                              // items [0, wide_n): a wavefront each
    int general_n, skip_first, skip_n;                    // items [wide_n, skip_first) and [skip_first + skip_n, n): a lane group each
    int short_first, short_n, single_first, single_n;     // whole segments with 2..kShortLen entries / with one entry
    int general_blocks, short_blocks;                     // blocks of the items before the short segments; of the short ones
    // destination-major
    const int32_t* in_pair;
    const void* KM;          // [P][2][D]
    const void* Q;           // [N][D]
    void* Z;                 // [N][D] (forward: written; backward: read)
    float2* ms;              // [N][H]
    float* partial;
    float2* part_ms;
    int piece_len;           // longest piece of a cut destination
    const void* dZ;          // [N][D]
    void* dQ;                // [N][D]
    float2* adl;             // [E][H] (att, dl)
    // pair-major
    const int32_t* out_epos;
    const int32_t* out_dst;
    void* dKM;               // [P][2][D]
};

// ------------------------------------------------------------------------------------------------ forward

// One batch of NE edges of an item: logits, running maximum, weighted sum.  The weights are not normalised yet, and a sum of n
// messages may exceed fp32 where their mean does not: acc carries the factor c = pow2_share(n), exact like its removal.
template <int V, int LPH, int NE>
struct FwdState {
    float m = -INFINITY, s = 0.f, c, acc[V];
    __device__ __forceinline__ explicit FwdState(float share) : c(share) { zero_cols(acc); }
    // the factor that makes acc the mean
    __device__ __forceinline__ float inverse() const { return 1.f / s * (1.f / c); }
    template <typename T>
    __device__ __forceinline__ void batch(const float (&q)[V], const rgnn_v4u (&k)[NE], const rgnn_v4u (&mr)[NE], int n) {
        float l[NE], mn = m;
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            float kv[V];
            widen_raw(k[u], kv);
            const float x = group_sum<LPH>(dot_cols(q, kv));
            l[u] = u < n ? x : -INFINITY;
            mn = fmaxf(mn, l[u]);
        }
        const float base = softmax_base(mn), sc = expf(m - base);     // 0 in the first batch (m = -inf), 1 while the maximum stands
        float t = 0.f;
#pragma unroll
        for (int c = 0; c < V; ++c) acc[c] *= sc;
        float p[NE];
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            p[u] = expf(l[u] - base);
            t += p[u];
            p[u] *= c;
        }
        add_rows<T>(acc, p, mr);
        s = s * sc + t;
        m = mn;
    }
};

// Whole destinations or pieces of cut ones, four edges (eight row loads) in flight per lane group, the pair ids one
// batch ahead.  NG lane groups share an item and take its batches in turn: one group for ordinary items, all groups of
// a wavefront for the long ones (at least kWideMin entries, so every group has edges), whose partial softmax states are
// merged at the end.  (A wavefront per long item reads and writes per-edge data in runs of 16 edges: the
// backward walk, which stores (att, dl), went from 2.58 to 2.46 ms at the sizes above, the forward from 2.03 to 2.01.)
template <int D, typename T, int LPH, int NG>
__device__ __forceinline__ void fwd_walk(const WalkArgs& a, int i) {
    constexpr int V = RowT<T>::V, LPR = D / V, H = LPR / LPH;
    const int cv = threadIdx.x % LPR, head = cv / LPH, sub = NG > 1 ? (threadIdx.x & 63) / LPR : 0;
    const T* __restrict__ KM = static_cast<const T*>(a.KM) + cv * V;
    const int b = a.it.beg[i], e = a.it.end[i], slot = a.it.slot[i];
    const size_t v = (size_t)a.it.row[i];
    FwdState<V, LPH, 4> f(slot < 0 ? pow2_share(e - b) : pow2_share(a.piece_len));
    if (b < e) {
        const int j0 = b + 4 * sub;
        int pr[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) pr[u] = a.in_pair[min(j0 + u, e - 1)];
        float q[V];
        load_cols(static_cast<const T*>(a.Q) + v * D + cv * V, q);
        for (int j = j0; j < e; j += 4 * NG) {
            rgnn_v4u k[4], m[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const T* p = KM + (size_t)pr[u] * 2 * D;
                k[u] = load_raw(p);
                m[u] = load_raw(p + D);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) pr[u] = a.in_pair[min(j + 4 * NG + u, e - 1)];
            f.template batch<T>(q, k, m, e - j);
        }
    }
    if (NG > 1) {
        float mn = f.m;
#pragma unroll
        for (int o = LPR; o < 64; o <<= 1) mn = fmaxf(mn, __shfl_xor(mn, o));
        const float sc = expf(f.m - softmax_base(mn));
        f.m = mn;
        f.s *= sc;
#pragma unroll
        for (int c = 0; c < V; ++c) f.acc[c] *= sc;
#pragma unroll
        for (int o = LPR; o < 64; o <<= 1) {
            f.s += __shfl_xor(f.s, o);
#pragma unroll
            for (int c = 0; c < V; ++c) f.acc[c] += __shfl_xor(f.acc[c], o);
        }
        if (sub != 0) return;
    }
    if (slot < 0) {
        const float inv = b < e ? f.inverse() : 0.f;      // a destination without edges gets the zero row
#pragma unroll
        for (int c = 0; c < V; ++c) f.acc[c] *= inv;
        store_cols(static_cast<T*>(a.Z) + v * D + cv * V, f.acc);
        if (cv % LPH == 0) a.ms[v * H + head] = make_float2(b < e ? f.m : 0.f, b < e ? f.s : 1.f);
    } else {
        store_cols(a.partial + (size_t)slot * D + cv * V, f.acc);
        if (cv % LPH == 0) a.part_ms[(size_t)slot * H + head] = make_float2(f.m, f.s);
    }
}
// index of this lane group's item among the ones a lane group takes alone, or -1
template <int LPR>
__device__ __forceinline__ int group_item(const WalkArgs& a) {
    const int k = (blockIdx.x - a.wide_blocks) * (256 / LPR) + threadIdx.x / LPR;
    if (k >= a.general_n) return -1;
    const int i = a.wide_n + k;
    return i >= a.skip_first ? i + a.skip_n : i;
}

// Whole destinations of at most NE edges, NI of them per lane group with all their loads independent: such a
// destination is a single batch, and alone it would leave the group waiting on its item -> pair -> row chain.
template <int D, typename T, int LPH, int NI, int NE>
__device__ __forceinline__ void fwd_few(const WalkArgs& a, int blk, int first, int n) {
    constexpr int V = RowT<T>::V, LPR = D / V, GPB = 256 / LPR, H = LPR / LPH;
    const int i0 = NI * (blk * GPB + threadIdx.x / LPR), cv = threadIdx.x % LPR, head = cv / LPH;
    if (i0 >= n) return;
    const T* __restrict__ KM = static_cast<const T*>(a.KM) + cv * V;
    int b[NI], e[NI], row[NI];
#pragma unroll
    for (int x = 0; x < NI; ++x) {
        const int i = first + min(i0 + x, n - 1);
        b[x] = a.it.beg[i];
        e[x] = a.it.end[i];
        row[x] = a.it.row[i];
    }
    rgnn_v4u k[NI][NE], m[NI][NE], q[NI];
#pragma unroll
    for (int x = 0; x < NI; ++x) q[x] = load_raw(static_cast<const T*>(a.Q) + (size_t)row[x] * D + cv * V);
    int pr[NI][NE];
#pragma unroll
    for (int x = 0; x < NI; ++x)
#pragma unroll
        for (int u = 0; u < NE; ++u) pr[x][u] = a.in_pair[min(b[x] + u, e[x] - 1)];
#pragma unroll
    for (int x = 0; x < NI; ++x)
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            const T* p = KM + (size_t)pr[x][u] * 2 * D;
            k[x][u] = load_raw(p);
            m[x][u] = load_raw(p + D);
        }
#pragma unroll
    for (int x = 0; x < NI; ++x) {
        if (i0 + x >= n) break;
        float qv[V];
        widen_raw(q[x], qv);
        FwdState<V, LPH, NE> f(pow2_share(e[x] - b[x]));
        f.template batch<T>(qv, k[x], m[x], e[x] - b[x]);
        const float inv = f.inverse();
#pragma unroll
        for (int c = 0; c < V; ++c) f.acc[c] *= inv;
        store_cols(static_cast<T*>(a.Z) + (size_t)row[x] * D + cv * V, f.acc);
        if (cv % LPH == 0) a.ms[(size_t)row[x] * H + head] = make_float2(f.m, f.s);
    }
}
// One launch for all items: the long ones first (a wavefront each), then the ordinary ones, then the short segments, which fill
// the machine while the long ones drain.  (Two launches cost 6 us of the 31 that 300k edges take, and a tail each.)
template <int D, typename T, int LPH>
__global__ __launch_bounds__(256) void hgt_attend_fwd_kernel(WalkArgs a) {
    constexpr int LPR = D / RowT<T>::V;
    const int blk = (int)blockIdx.x - a.general_blocks;
    if ((int)blockIdx.x < a.wide_blocks) {
        const int i = blockIdx.x * 4 + threadIdx.x / 64;
        if (i < a.wide_n) fwd_walk<D, T, LPH, 64 / LPR>(a, i);
    } else if (blk < 0) {
        const int i = group_item<LPR>(a);
        if (i >= 0) fwd_walk<D, T, LPH, 1>(a, i);
    } else if (blk < a.short_blocks) fwd_few<D, T, LPH, 2, kShortLen>(a, blk, a.short_first, a.short_n);
    else fwd_few<D, T, LPH, 4, 1>(a, blk - a.short_blocks, a.single_first, a.single_n);
}

// ------------------------------------------------------------------------------------------------ backward, destination-major

// One batch of NE edges (n of them exist): dq += dl Ka; lane t of a head's LPH lanes keeps (att, dl) of the edges t, t + LPH, ...
// of the batch in `mine`.
template <typename T, int V, int LPH, int NE>
struct BwdBatch {
    static constexpr int NS = (NE + LPH - 1) / LPH;
    float2 mine[NS];
    __device__ __forceinline__ void form(const float (&q)[V], const float (&gz)[V], float gbar, float2 ms, float inv,
                                         const rgnn_v4u (&k)[NE], const rgnn_v4u (&mr)[NE], int n, int t, float (&dq)[V]) {
        float dl[NE];
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            float kv[V], mv[V];
            widen_raw(k[u], kv);
            widen_raw(mr[u], mv);
            const float l = group_sum<LPH>(dot_cols(q, kv));
            const float g = group_sum<LPH>(dot_cols(gz, mv));
            const float att = expf(l - ms.x) * inv;
            dl[u] = u < n ? att * (g - gbar) : 0.f;
            if (t == u % LPH) mine[u / LPH] = make_float2(att, dl[u]);
        }
        add_rows<T>(dq, dl, k);
    }
    // adl: the entry of the batch's first edge and this lane's head; the lanes of a group fill whole lines
    __device__ __forceinline__ void store(float2* __restrict__ adl, int n, int H, int t) const {
#pragma unroll
        for (int x = 0; x < NS; ++x)
            if (t + x * LPH < NE && t + x * LPH < n) adl[(size_t)(t + x * LPH) * H] = mine[x];
    }
};

template <int D, typename T, int LPH, int NG>
__device__ __forceinline__ void bwd_walk(const WalkArgs& a, int i) {
    constexpr int V = RowT<T>::V, LPR = D / V, H = LPR / LPH;
    const int cv = threadIdx.x % LPR, head = cv / LPH, t = cv % LPH, sub = NG > 1 ? (threadIdx.x & 63) / LPR : 0;
    const T* __restrict__ KM = static_cast<const T*>(a.KM) + cv * V;
    const int b = a.it.beg[i], e = a.it.end[i], slot = a.it.slot[i];
    const size_t v = (size_t)a.it.row[i];
    float dq[V];
    zero_cols(dq);
    if (b < e) {
        const int j0 = b + 4 * sub;
        int pr[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) pr[u] = a.in_pair[min(j0 + u, e - 1)];
        float q[V], gz[V], zz[V];
        load_cols(static_cast<const T*>(a.Q) + v * D + cv * V, q);
        load_cols(static_cast<const T*>(a.dZ) + v * D + cv * V, gz);
        load_cols(static_cast<const T*>(a.Z) + v * D + cv * V, zz);
        const float2 ms = a.ms[v * H + head];
        const float gbar = group_sum<LPH>(dot_cols(gz, zz)), inv = 1.f / ms.y;
        // A batch's (att, dl) leave after the next batch's rows have been asked for: loads and stores complete in issue
        // order, so a store issued before the loads would have to be acknowledged before the rows can be used.
        BwdBatch<T, V, LPH, 4> batch;
        float2* adl = a.adl + (size_t)b * H + head;
        int j = j0;
        for (; j < e; j += 4 * NG) {
            rgnn_v4u k[4], m[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const T* p = KM + (size_t)pr[u] * 2 * D;
                k[u] = load_raw(p);
                m[u] = load_raw(p + D);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) pr[u] = a.in_pair[min(j + 4 * NG + u, e - 1)];
            __builtin_amdgcn_sched_barrier(0);
            if (j > j0) batch.store(adl + (size_t)(j - 4 * NG - b) * H, 4, H, t);
            batch.form(q, gz, gbar, ms, inv, k, m, e - j, t, dq);
        }
        j -= 4 * NG;
        batch.store(adl + (size_t)(j - b) * H, e - j, H, t);
    }
    if (NG > 1) {
#pragma unroll
        for (int o = LPR; o < 64; o <<= 1)
#pragma unroll
            for (int c = 0; c < V; ++c) dq[c] += __shfl_xor(dq[c], o);
        if (sub != 0) return;
    }
    if (slot < 0) store_cols(static_cast<T*>(a.dQ) + v * D + cv * V, dq);
    else store_cols(a.partial + (size_t)slot * D + cv * V, dq);
}

template <int D, typename T, int LPH, int NI, int NE>
__device__ __forceinline__ void bwd_few(const WalkArgs& a, int blk, int first, int n) {
    constexpr int V = RowT<T>::V, LPR = D / V, GPB = 256 / LPR, H = LPR / LPH;
    const int i0 = NI * (blk * GPB + threadIdx.x / LPR), cv = threadIdx.x % LPR, head = cv / LPH, t = cv % LPH;
    if (i0 >= n) return;
    const T* __restrict__ KM = static_cast<const T*>(a.KM) + cv * V;
    int b[NI], e[NI], row[NI];
#pragma unroll
    for (int x = 0; x < NI; ++x) {
        const int i = first + min(i0 + x, n - 1);
        b[x] = a.it.beg[i];
        e[x] = a.it.end[i];
        row[x] = a.it.row[i];
    }
    int pr[NI][NE];
#pragma unroll
    for (int x = 0; x < NI; ++x)
#pragma unroll
        for (int u = 0; u < NE; ++u) pr[x][u] = a.in_pair[min(b[x] + u, e[x] - 1)];
    rgnn_v4u q[NI], gz[NI], zz[NI];
    float2 ms[NI];
#pragma unroll
    for (int x = 0; x < NI; ++x) {
        const size_t at = (size_t)row[x] * D + cv * V;
        q[x] = load_raw(static_cast<const T*>(a.Q) + at);
        gz[x] = load_raw(static_cast<const T*>(a.dZ) + at);
        zz[x] = load_raw(static_cast<const T*>(a.Z) + at);
        ms[x] = a.ms[(size_t)row[x] * H + head];
    }
    rgnn_v4u k[NI][NE], m[NI][NE];
#pragma unroll
    for (int x = 0; x < NI; ++x)
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            const T* p = KM + (size_t)pr[x][u] * 2 * D;
            k[x][u] = load_raw(p);
            m[x][u] = load_raw(p + D);
        }
#pragma unroll
    for (int x = 0; x < NI; ++x) {
        if (i0 + x >= n) break;
        float qv[V], gv[V], zv[V], dq[V];
        widen_raw(q[x], qv);
        widen_raw(gz[x], gv);
        widen_raw(zz[x], zv);
        zero_cols(dq);
        const float gbar = group_sum<LPH>(dot_cols(gv, zv));
        BwdBatch<T, V, LPH, NE> batch;
        batch.form(qv, gv, gbar, ms[x], 1.f / ms[x].y, k[x], m[x], e[x] - b[x], t, dq);
        batch.store(a.adl + (size_t)b[x] * H + head, e[x] - b[x], H, t);
        store_cols(static_cast<T*>(a.dQ) + (size_t)row[x] * D + cv * V, dq);
    }
}
template <int D, typename T, int LPH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void hgt_attend_bwd_kernel(WalkArgs a) {
    constexpr int LPR = D / RowT<T>::V;
    const int blk = (int)blockIdx.x - a.general_blocks;
    if ((int)blockIdx.x < a.wide_blocks) {
        const int i = blockIdx.x * 4 + threadIdx.x / 64;
        if (i < a.wide_n) bwd_walk<D, T, LPH, 64 / LPR>(a, i);
    } else if (blk < 0) {
        const int i = group_item<LPR>(a);
        if (i >= 0) bwd_walk<D, T, LPH, 1>(a, i);
    } else if (blk < a.short_blocks) bwd_few<D, T, LPH, 2, kShortLen>(a, blk, a.short_first, a.short_n);
    else bwd_few<D, T, LPH, 4, 1>(a, blk - a.short_blocks, a.single_first, a.single_n);
}

// ------------------------------------------------------------------------------------------------ backward, pair-major

template <int D, typename T, int LPH>
__device__ __forceinline__ void pair_walk(const WalkArgs& a, int i) {
    constexpr int V = RowT<T>::V, LPR = D / V, H = LPR / LPH;
    const int cv = threadIdx.x % LPR, head = cv / LPH;
    const T* __restrict__ Q = static_cast<const T*>(a.Q) + cv * V;
    const T* __restrict__ dZ = static_cast<const T*>(a.dZ) + cv * V;
    const int b = a.it.beg[i], e = a.it.end[i], slot = a.it.slot[i];
    float dk[V], dm[V];
    zero_cols(dk);
    zero_cols(dm);
    // indices and coefficients run one batch ahead of the rows; positions past the end repeat the last entry with
    // zero coefficients
    int row[4];
    float2 c[4];
    auto fetch = [&](int j) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int jj = min(j + u, e - 1);
            row[u] = a.out_dst[jj];
            c[u] = a.adl[(size_t)a.out_epos[jj] * H + head];
            if (j + u >= e) c[u] = make_float2(0.f, 0.f);
        }
    };
    if (b < e) fetch(b);
    for (int j = b; j < e; j += 4) {
        rgnn_v4u q[4], z[4];
        float att[4], dl[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            q[u] = load_raw(Q + (size_t)row[u] * D);
            z[u] = load_raw(dZ + (size_t)row[u] * D);
            att[u] = c[u].x;
            dl[u] = c[u].y;
        }
        if (j + 4 < e) fetch(j + 4);
        add_rows<T>(dk, dl, q);
        add_rows<T>(dm, att, z);
    }
    if (slot < 0) {
        T* o = static_cast<T*>(a.dKM) + (size_t)a.it.row[i] * 2 * D + cv * V;
        store_cols(o, dk);
        store_cols(o + D, dm);
    } else {
        float* o = a.partial + (size_t)slot * 2 * D + cv * V;
        store_cols(o, dk);
        store_cols(o + D, dm);
    }
}

template <int D, typename T, int LPH, int NI, int NE>
__device__ __forceinline__ void pair_few(const WalkArgs& a, int blk, int first, int n) {
    constexpr int V = RowT<T>::V, LPR = D / V, GPB = 256 / LPR, H = LPR / LPH;
    const int i0 = NI * (blk * GPB + threadIdx.x / LPR), cv = threadIdx.x % LPR, head = cv / LPH;
    if (i0 >= n) return;
    const T* __restrict__ Q = static_cast<const T*>(a.Q) + cv * V;
    const T* __restrict__ dZ = static_cast<const T*>(a.dZ) + cv * V;
    int b[NI], e[NI], orow[NI];
#pragma unroll
    for (int x = 0; x < NI; ++x) {
        const int i = first + min(i0 + x, n - 1);
        b[x] = a.it.beg[i];
        e[x] = a.it.end[i];
        orow[x] = a.it.row[i];
    }
    int row[NI][NE], at[NI][NE];
#pragma unroll
    for (int x = 0; x < NI; ++x)
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            const int jj = min(b[x] + u, e[x] - 1);
            row[x][u] = a.out_dst[jj];
            at[x][u] = a.out_epos[jj];
        }
    rgnn_v4u q[NI][NE], z[NI][NE];
    float2 c[NI][NE];
#pragma unroll
    for (int x = 0; x < NI; ++x)
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            q[x][u] = load_raw(Q + (size_t)row[x][u] * D);
            z[x][u] = load_raw(dZ + (size_t)row[x][u] * D);
            c[x][u] = a.adl[(size_t)at[x][u] * H + head];
        }
#pragma unroll
    for (int x = 0; x < NI; ++x) {
        if (i0 + x >= n) break;
        float dk[V], dm[V];
        zero_cols(dk);
        zero_cols(dm);
        float att[NE], dl[NE];
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            const bool ok = b[x] + u < e[x];
            att[u] = ok ? c[x][u].x : 0.f;
            dl[u] = ok ? c[x][u].y : 0.f;
        }
        add_rows<T>(dk, dl, q[x]);
        add_rows<T>(dm, att, z[x]);
        T* o = static_cast<T*>(a.dKM) + (size_t)orow[x] * 2 * D + cv * V;
        store_cols(o, dk);
        store_cols(o + D, dm);
    }
}
template <int D, typename T, int LPH>
__global__ __launch_bounds__(256) void hgt_pair_bwd_kernel(WalkArgs a) {
    const int blk = (int)blockIdx.x - a.general_blocks;
    if (blk < 0) {
        const int i = group_item<D / RowT<T>::V>(a);
        if (i >= 0) pair_walk<D, T, LPH>(a, i);
    } else if (blk < a.short_blocks) pair_few<D, T, LPH, 2, kShortLen>(a, blk, a.short_first, a.short_n);
    else pair_few<D, T, LPH, 4, 1>(a, blk - a.short_blocks, a.single_first, a.single_n);
}

// Fills the item ranges of a walk over L; returns its number of blocks.
int split_ranges(const ItemList& L, int groups_per_block, bool wide, WalkArgs& a) {
    const int ns = batched_count(L.num_single, current_schedule_flags());
    const int nsh = batched_count(L.num_short, current_schedule_flags());
    a.it = dev_items(L);
    a.wide_n = wide ? L.num_wide : 0;
    a.wide_blocks = (int)blocks_for((size_t)a.wide_n, 4);
    a.general_n = L.num_items - a.wide_n - nsh - ns;
    a.skip_first = nsh > 0 ? L.first_short : L.first_single;
    a.skip_n = nsh + ns;
    a.short_first = L.first_short; a.short_n = nsh;
    a.single_first = L.first_single; a.single_n = ns;
    a.short_blocks = nsh > 0 ? (int)blocks_for((size_t)(nsh + 1) / 2, groups_per_block) : 0;
    a.general_blocks = a.wide_blocks + (int)blocks_for((size_t)a.general_n, groups_per_block);
    return a.general_blocks + a.short_blocks + (ns > 0 ? (int)blocks_for((size_t)(ns + 3) / 4, groups_per_block) : 0);
}

}  // namespace

// Runs the statement with DD = width, TT = row type and LL = lanes per head.  Heads are 16, 32 or 64 columns wide.
#define RGNN_HGT_LPH(DD_, T_, LPH_, ...)                                                           \
    do {                                                                                           \
        constexpr int DD = DD_;                                                                    \
        using TT = T_;                                                                             \
        if ((LPH_) == 4) { constexpr int LL = 4; __VA_ARGS__; }                                    \
        else if ((LPH_) == 8) { constexpr int LL = 8; __VA_ARGS__; }                               \
        else if (sizeof(T_) == 2 && (LPH_) == 2) { constexpr int LL = sizeof(T_) == 2 ? 2 : 4; __VA_ARGS__; }        \
        else if (sizeof(T_) == 4 && DD_ >= 64 && (LPH_) == 16) { constexpr int LL = sizeof(T_) == 4 && DD_ >= 64 ? 16 : 4; __VA_ARGS__; } \
        else RGNN_FAIL(RGNN_EUNSUPPORTED, "HGT walk: width %d with %d lanes per head is not built", DD_, (int)(LPH_)); \
    } while (0)
#define RGNN_HGT_DISPATCH(D_, H_, B16_, ...)                                                       \
    do {                                                                                           \
        const int lph_ = (D_) / ((B16_) ? 8 : 4) / (H_);                                           \
        if (B16_) {                                                                                \
            if ((D_) != 128) RGNN_FAIL(RGNN_EUNSUPPORTED, "bf16 rows need width 128, got %d", (int)(D_)); \
            RGNN_HGT_LPH(128, bf16_t, lph_, __VA_ARGS__);                                          \
        } else if ((D_) == 128) RGNN_HGT_LPH(128, float, lph_, __VA_ARGS__);                       \
        else if ((D_) == 64) RGNN_HGT_LPH(64, float, lph_, __VA_ARGS__);                           \
        else if ((D_) == 32) RGNN_HGT_LPH(32, float, lph_, __VA_ARGS__);                           \
        else RGNN_FAIL(RGNN_EUNSUPPORTED, "feature width %d not supported (32/64/128)", (int)(D_)); \
    } while (0)

#define RGNN_HGT_WALK(KERNEL, WIDE)                                                                                              \
    do {                                                                                                                          \
        const int blocks = split_ranges(L, 256 / (D / (rows_bf16 ? 8 : 4)), WIDE, a);                                              \
        RGNN_HGT_DISPATCH(D, H, rows_bf16, hipLaunchKernelGGL((KERNEL##_kernel<DD, TT, LL>), dim3(blocks), dim3(256), 0, st, a));  \
        RGNN_CHECK_LAUNCH();                                                                                                      \
    } while (0)

rgnn_status_t hgt_attend_fwd(const rgnn_graph* g, int D, int H, const void* KM, const void* Q, void* Z, float* ms,
                             float* partial, float* part_ms, hipStream_t st, int rows_bf16) {
    const ItemList& L = g->dst_items;
    if (L.num_items == 0) return RGNN_OK;
    WalkArgs a{};
    a.in_pair = g->idx[RGNN_IDX_IN_PAIR]; a.KM = KM; a.Q = Q; a.Z = Z; a.ms = reinterpret_cast<float2*>(ms);
    a.partial = partial; a.part_ms = reinterpret_cast<float2*>(part_ms); a.piece_len = item_cut(g->E);
    {
        KernelTimer kt(st, "hgt_attend_fwd");
        RGNN_HGT_WALK(hgt_attend_fwd, true);
    }
    return combine_softmax(L, D, H, partial, part_ms, Z, rows_bf16, ms, true, a.piece_len, "hgt_attend_fwd.combine", st);
}

rgnn_status_t hgt_attend_bwd(const rgnn_graph* g, int D, int H, const void* KM, const void* Q, const void* Z, const float* ms,
                             const void* dZ, void* dQ, float* adl, float* partial, hipStream_t st, int rows_bf16) {
    const ItemList& L = g->dst_items;
    if (L.num_items == 0) return RGNN_OK;
    WalkArgs a{};
    a.in_pair = g->idx[RGNN_IDX_IN_PAIR]; a.KM = KM; a.Q = Q; a.Z = const_cast<void*>(Z);
    a.ms = reinterpret_cast<float2*>(const_cast<float*>(ms)); a.partial = partial; a.dZ = dZ; a.dQ = dQ;
    a.adl = reinterpret_cast<float2*>(adl);
    {
        KernelTimer kt(st, "hgt_attend_bwd");
        RGNN_HGT_WALK(hgt_attend_bwd, true);
    }
    return combine_partials(L, D, partial, dQ, rows_bf16, "hgt_attend_bwd.combine", st);
}

rgnn_status_t hgt_pair_bwd(const rgnn_graph* g, int D, int H, const void* Q, const void* dZ, const float* adl, void* dKM,
                           float* partial, hipStream_t st, int rows_bf16) {
    const ItemList& L = g->pair_items;
    if (L.num_items == 0) return RGNN_OK;
    WalkArgs a{};
    a.Q = Q; a.dZ = dZ; a.adl = reinterpret_cast<float2*>(const_cast<float*>(adl)); a.dKM = dKM; a.partial = partial;
    a.out_epos = g->idx[RGNN_IDX_OUT_EPOS]; a.out_dst = g->idx[RGNN_IDX_OUT_DST];
    {
        KernelTimer kt(st, "hgt_pair_bwd");
        RGNN_HGT_WALK(hgt_pair_bwd, false);
    }
    return combine_partials(L, 2 * D, partial, dKM, rows_bf16, "hgt_pair_bwd.combine", st);
}

}  // namespace rgnn
