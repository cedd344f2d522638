// Edge-traversal kernels: per-destination edge softmax, weighted gather-sum aggregation
// (forward over destination-major CSR, backward over the pair-major transpose), the
// backward per-edge dot product, and the small segment sums around them.
//
// These replace the thesis's traversal template (Ch.3 "The GEMM Template and the Traversal
// Template": one block per edge or node, partial sums per thread and warp, then atomicAdd)
// by segment walks: every output row has exactly one owner, so nothing is accumulated with
// atomics and results do not depend on scheduling.  All of them are HBM-bound: a feature
// row of D floats is read by D/4 lanes as one 16-byte load each, so a 64-lane wavefront
// has four 256-byte rows (D = 64) in flight per load instruction, and the edge loop is
// unrolled four times to keep sixteen row reads in flight per wavefront.
//
// Segments longer than kItemMax entries (hub nodes) are cut into items by the graph index;
// an item of a cut segment writes a partial row and a combine kernel sums the partial rows
// of each cut segment in order.
#include "rgnn_internal.h"
#include "traversal.h"
#include "device_utils.h"
#include "schedule.h"

namespace rgnn {

static thread_local uint32_t g_schedule_flags = 0;
uint32_t current_schedule_flags() { return g_schedule_flags; }
ScheduleFlagsScope::ScheduleFlagsScope(uint32_t flags) : prev(g_schedule_flags) { g_schedule_flags = flags; }
ScheduleFlagsScope::~ScheduleFlagsScope() { g_schedule_flags = prev; }

// ------------------------------------------------------------------ small dense helpers

__global__ __launch_bounds__(256) void fold_weight_kernel(FoldArgs f) { fold_weight_block(f, blockIdx.x); }

// out[i * ostride + h] = sum_{j in [ptr[i], ptr[i+1])} val[(via ? via[j] : j) * stride + off + h],  h < heads.
// One launch: the first n_long * heads workgroups take one (long segment, head) each (segments of more
// than kSerialMax entries, listed by the graph index; the hub runs are thousands of entries long), the
// others one lane per (segment, head) for the segments up to that length.  The long ones come first so
// that the few workgroups that walk a hub run start at once and the short segments fill the machine
// around them.  The last `fold.blocks` workgroups fold weights (RGAT's backward: the two do not depend on each other, and a
// launch that is over in two microseconds costs five in a row of dependent ones).
__global__ __launch_bounds__(256) void segment_scalar_sum_kernel(FoldArgs fold, int n, int heads, const int32_t* __restrict__ ptr,
                                                                 const int32_t* __restrict__ via,
                                                                 const float* __restrict__ val, int stride, int off,
                                                                 int min_len, float* __restrict__ out, int n_long,
                                                                 const int32_t* __restrict__ long_ids, int ostride) {
    __shared__ float red[4];
    const int rest = (int)gridDim.x - fold.blocks;
    if ((int)blockIdx.x >= rest) {
        fold_weight_block(fold, blockIdx.x - rest);
        return;
    }
    const int lh = 31 - __clz(heads);            // the head count is a power of two (checked by the launcher)
    const int long_blocks = n_long << lh;
    if ((int)blockIdx.x < long_blocks) {
        // four loads in flight per lane, lane sums added in lane order, then the four wavefronts' sums in order
        const int i = long_ids[blockIdx.x >> lh], h = blockIdx.x & (heads - 1);
        const int b = ptr[i], e = ptr[i + 1];
        float t0 = 0.f, t1 = 0.f, t2 = 0.f, t3 = 0.f;
        for (int j = b + (int)threadIdx.x; j < e; j += 1024) {
            const int j1 = j + 256, j2 = j + 512, j3 = j + 768;
            t0 += val[(size_t)(via ? via[j] : j) * stride + off + h];
            if (j1 < e) t1 += val[(size_t)(via ? via[j1] : j1) * stride + off + h];
            if (j2 < e) t2 += val[(size_t)(via ? via[j2] : j2) * stride + off + h];
            if (j3 < e) t3 += val[(size_t)(via ? via[j3] : j3) * stride + off + h];
        }
        const float t = group_sum<64>((t0 + t1) + (t2 + t3));
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
        __syncthreads();
        if (threadIdx.x == 0) out[(size_t)i * ostride + h] = (red[0] + red[1]) + (red[2] + red[3]);
        return;
    }
    const int64_t t = (int64_t)(blockIdx.x - long_blocks) * 256 + threadIdx.x;
    if (t >= (int64_t)n * heads) return;
    const int i = (int)(t >> lh), h = (int)(t & (heads - 1));
    const int b = ptr[i], e = ptr[i + 1];
    if (e - b > kSerialMax || e - b < min_len) return;
    // four entries per step, every load unconditional (positions past the end repeat the last entry and
    // add zero), so that a lane has four values in flight instead of one; the sum keeps the entry order
    float s = 0.f;
    for (int j = b; j < e; j += 4) {
        int id[4];
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int jj = min(j + u, e - 1);
            id[u] = via ? via[jj] : jj;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = val[(size_t)id[u] * stride + off + h];
#pragma unroll
        for (int u = 0; u < 4; ++u) s += j + u < e ? v[u] : 0.f;
    }
    out[(size_t)i * ostride + h] = s;
}

// The same sums for HV = 2 or 4 heads whose values lie side by side (stride, off and ostride multiples of HV, val
// and out aligned to HV floats): one lane per segment adds all HV heads at once with vector loads, one workgroup per
// long segment.  The order of the additions per head is the one of the kernel above.
template <int HV>
__global__ __launch_bounds__(256) void segment_vec_sum_kernel(FoldArgs fold, int n, const int32_t* __restrict__ ptr,
                                                              const int32_t* __restrict__ via, const float* __restrict__ val,
                                                              int stride, int off, int min_len, float* __restrict__ out,
                                                              int n_long, const int32_t* __restrict__ long_ids, int ostride) {
    struct __align__(4 * HV) Vec { float v[HV]; };
    __shared__ float red[4][HV];
    const int rest = (int)gridDim.x - fold.blocks;
    if ((int)blockIdx.x >= rest) {
        fold_weight_block(fold, blockIdx.x - rest);
        return;
    }
    auto load = [&](int j) { return *reinterpret_cast<const Vec*>(val + (size_t)(via ? via[j] : j) * stride + off); };
    if ((int)blockIdx.x < n_long) {
        const int i = long_ids[blockIdx.x];
        const int b = ptr[i], e = ptr[i + 1];
        float t[4][HV];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int h = 0; h < HV; ++h) t[u][h] = 0.f;
        for (int j = b + (int)threadIdx.x; j < e; j += 1024) {
            Vec x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = load(min(j + 256 * u, e - 1));
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int h = 0; h < HV; ++h) t[u][h] += j + 256 * u < e ? x[u].v[h] : 0.f;
        }
#pragma unroll
        for (int h = 0; h < HV; ++h) {
            const float w = group_sum<64>((t[0][h] + t[1][h]) + (t[2][h] + t[3][h]));
            if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][h] = w;
        }
        __syncthreads();
        if (threadIdx.x < HV) out[(size_t)i * ostride + threadIdx.x] = (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
        return;
    }
    const int64_t i = (int64_t)(blockIdx.x - n_long) * 256 + threadIdx.x;
    if (i >= n) return;
    const int b = ptr[i], e = ptr[i + 1];
    if (e - b > kSerialMax || e - b < min_len) return;
    Vec s;
#pragma unroll
    for (int h = 0; h < HV; ++h) s.v[h] = 0.f;
    for (int j = b; j < e; j += 4) {
        Vec x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = load(min(j + u, e - 1));
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int h = 0; h < HV; ++h) s.v[h] += j + u < e ? x[u].v[h] : 0.f;
    }
    *reinterpret_cast<Vec*>(out + (size_t)i * ostride) = s;
}

// ------------------------------------------------------------------ edge softmax (RGAT)

// Per item of the destination-major list: l_e = leakyrelu(s_src[pair] + s_dst[run]) is
// written to att, then max and sum of exp; a whole-node item normalises at once
// (att_e = +-exp(l - m)/sum, sign bit set when z_e <= 0), a piece of a cut node stores
// (m, sum) for the combine step.
struct SoftmaxArgs {
    Items it;
    const int32_t* in_pair;
    const int32_t* in_run;
    const float* s_src;
    const float* s_dst;
    float slope;
    float* att;
    float* part_m;
    float* part_s;
    float2* ms;      // optional [N]: (max, sum of exp) of every destination with edges
};

__device__ __forceinline__ float signed_att(float l, float m, float inv) {
    const float a = expf(l - m) * inv;
    return l > 0.f ? a : -a;
}

// Destinations with at most kSerialMax incoming edges: one lane per node, in node order, so
// that neighbouring lanes walk neighbouring CSR ranges.  The logits stay in registers (the loop
// over the kSerialMax slots is fully unrolled and predicated), eight index pairs and then eight
// logit gathers are in flight at a time, and att is written once.  Everything else (longer nodes
// and the pieces of cut nodes) goes through edge_softmax_long_kernel.
__global__ __launch_bounds__(256) void edge_softmax_kernel(SoftmaxArgs a, int N, const int32_t* __restrict__ in_ptr) {
    const int v = blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    const int b = in_ptr[v], len = in_ptr[v + 1] - b;
    if (len == 0 || len > kSerialMax) return;
    float l[kSerialMax];
#pragma unroll
    for (int c = 0; c < kSerialMax; c += 8) {
        if (c < len) {
            int pr[8], rn[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int j = b + min(c + u, len - 1);
                pr[u] = a.in_pair[j];
                rn[u] = a.in_run[j];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float z = a.s_src[pr[u]] + a.s_dst[rn[u]];
                l[c + u] = c + u < len ? (z > 0.f ? z : a.slope * z) : -INFINITY;
            }
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) l[c + u] = -INFINITY;
        }
    }
    float m = -INFINITY, s = 0.f;
#pragma unroll
    for (int k = 0; k < kSerialMax; ++k) m = fmaxf(m, l[k]);
#pragma unroll
    for (int k = 0; k < kSerialMax; ++k) s += expf(l[k] - m);     // the empty slots add exp(-inf) = 0
    const float inv = 1.f / s;
#pragma unroll
    for (int k = 0; k < kSerialMax; ++k)
        if (k < len) a.att[b + k] = signed_att(l[k], m, inv);
    if (a.ms) a.ms[v] = make_float2(m, s);
}

// One wavefront per item that is longer than kSerialMax or is a piece of a cut node.  An item has at
// most kItemMax entries, kItemMax / 64 per lane, which stay in registers between the passes.
__global__ __launch_bounds__(256) void edge_softmax_long_kernel(SoftmaxArgs a, int n_long, const int32_t* __restrict__ long_item) {
    constexpr int PER = kItemMax / 64;
    const int w = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (w >= n_long) return;
    const int i = long_item[w];
    const int bb = a.it.beg[i], ee = a.it.end[i], sl = a.it.slot[i];
    float l[PER];
    int pr[PER], rn[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int j = min(bb + lane + 64 * u, ee - 1);
        pr[u] = a.in_pair[j];
        rn[u] = a.in_run[j];
    }
    float m = -INFINITY, s = 0.f;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const float z = a.s_src[pr[u]] + a.s_dst[rn[u]];
        l[u] = bb + lane + 64 * u < ee ? (z > 0.f ? z : a.slope * z) : -INFINITY;
        m = fmaxf(m, l[u]);
    }
    m = wave_max(m);
#pragma unroll
    for (int u = 0; u < PER; ++u) s += expf(l[u] - m);
    s = group_sum<64>(s);
    if (sl < 0) {
        const float inv = 1.f / s;
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (bb + lane + 64 * u < ee) a.att[bb + lane + 64 * u] = signed_att(l[u], m, inv);
        if (a.ms && lane == 0) a.ms[a.it.row[i]] = make_float2(m, s);
    } else {
        // a piece of a cut node: the finish kernel normalises, from the logits
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (bb + lane + 64 * u < ee) a.att[bb + lane + 64 * u] = l[u];
        if (lane == 0) {
            a.part_m[sl] = m;
            a.part_s[sl] = s;
        }
    }
}

// Cut nodes: combine the pieces' (m, sum) in order, then normalise every piece.
// One wavefront per piece; each recomputes its node's totals (a node has few pieces).
__global__ void edge_softmax_finish_kernel(int num_partials, const int32_t* __restrict__ part_item,
                                           const int32_t* __restrict__ part_split,
                                           const int32_t* __restrict__ split_ptr, Items it,
                                           const float* __restrict__ part_m, const float* __restrict__ part_s,
                                           float* __restrict__ att, float2* __restrict__ ms) {
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= num_partials) return;
    const int sp = part_split[t];
    const int p0 = split_ptr[sp], p1 = split_ptr[sp + 1];
    float m = -INFINITY;
    for (int p = p0 + lane; p < p1; p += 64) m = fmaxf(m, part_m[p]);
    m = wave_max(m);
    float s = 0.f;
    for (int p = p0 + lane; p < p1; p += 64) s += part_s[p] * expf(part_m[p] - m);
    s = group_sum<64>(s);
    const float inv = 1.f / s;
    const int item = part_item[t];
    for (int j = it.beg[item] + lane; j < it.end[item]; j += 64) att[j] = signed_att(att[j], m, inv);
    if (ms && t == p0 && lane == 0) ms[it.row[item]] = make_float2(m, s);     // the node's first piece records its totals
}

// ------------------------------------------------------------------ weighted gather-sum

// For item i with entries j in [beg, end):
//   k   = via ? via[j] : j
//   row = rowidx ? (row_by_k ? rowidx[k] : rowidx[j]) : k
//   c   = coef ? coef[k * cstride + head] : 1     (absolute value if cabs; head = which of the
//                                                  `heads` equal column groups the lane's columns lie in)
//   acc += c * src[row]
// and acc goes to out[row_i] (whole segment) or partial[slot] (piece of a cut segment).
struct GatherArgs {
    Items it;
    const int32_t* via;
    const int32_t* rowidx;
    int row_by_k;
    const float* coef;
    int cstride;
    int cabs;
    int lanes_per_head;   // lanes per row / heads
    const void* src;      // rows of TI
    void* out;            // rows of TO
    float* partial;       // fp32 rows
    int skip_first;       // items [skip_first, skip_first + skip_n) are left to the short-segment and single-entry walks
    int skip_n;
    Rank1 r1;             // optional: out[row_i] += r1.coef[row_i][head] * r1.vec[r1.seg[row_i]] (whole segments here,
                          // cut segments when their pieces are combined)
    float* sum2;          // optional (S2 kernels): sum2[row_i * sum2_stride + head] = sum_j coef[k * cstride + s2off + head]
    int sum2_stride;      // for the whole segments, added in entry order; the caller sums the cut segments itself.  With
    int s2off;            // r1.vec set, the walk also adds that sum times r1.vec[r1.seg[row_i]] to the row (r1.coef then
                          // serves only the cut segments, where their pieces are combined)
    const float* extra;   // optional (EX kernels): out[row_i] += extra[row_i] (cut segments: where their pieces are combined); may be out
};

// the rank-1 term of a whole segment whose coefficient the walk has just summed
template <int D, int V>
__device__ __forceinline__ void add_rank1_own(const Rank1& r1, float c, size_t row, int cv, float (&acc)[V]) {
    if (!r1.vec) return;
    float t[V];
    load_cols(r1.vec + (size_t)r1.seg[row] * D + cv * V, t);
    fma_cols(acc, c, t);
}

template <int D, int V>
__device__ __forceinline__ void add_row(const float* extra, size_t row, int cv, float (&acc)[V]) {
    if (!extra) return;
    float t[V];
    load_cols(extra + row * D + cv * V, t);
    fma_cols(acc, 1.f, t);
}
template <int D, int V>
__device__ __forceinline__ void add_rank1(const Rank1& r1, int lanes_per_head, size_t row, int cv, float (&acc)[V]) {
    if (!r1.coef) return;
    const float c = r1.coef[row * r1.stride + cv / lanes_per_head];
    float t[V];
    load_cols(r1.vec + (size_t)r1.seg[row] * D + cv * V, t);
    fma_cols(acc, c, t);
}

// ROLE gives each use its own kernel name in profiler output (0 forward aggregation over destinations,
// 1 backward aggregation over pairs, 2 destination-side weight gradient, 3 gradient rows of the runs over sources, plus a row).  The forward aggregation
// gathers rows of the large per-pair tensor, most of them once: with fp32 rows those loads carry the
// non-temporal hint (NT; it did not pay for the 2-byte rows, whose pairs are shared by more edges in the
// workloads that use them); the other two gather rows of node tensors, which are reused and stay cached.
// TI / TO: storage type of the gathered rows and of the output rows (float or bf16_t).
template <int D, typename TI, typename TO, bool R1, bool NT, bool S2 = false, bool EX = false>
__device__ __forceinline__ void gather_general(const GatherArgs& a, int blk) {
    constexpr int V = RowT<TI>::V, LPR = D / V, IPB = 256 / LPR;
    int i = blk * IPB + threadIdx.x / LPR;
    const int cv = threadIdx.x % LPR;
    if (i >= a.it.n - a.skip_n) return;
    if (i >= a.skip_first) i += a.skip_n;      // the single-entry segments have their own kernel
    const TI* __restrict__ src = static_cast<const TI*>(a.src);
    const int b = a.it.beg[i], e = a.it.end[i];
    const int head = cv / a.lanes_per_head;
    float acc0[V], acc1[V];
    zero_cols(acc0);
    zero_cols(acc1);
    // Indices and coefficients run one batch of four ahead of the rows, so that a batch costs one
    // memory round trip instead of two.  Positions past the end repeat the last entry with a zero
    // coefficient: every load is unconditional.
    int row[4];
    float c[4], c2[S2 ? 4 : 1], s2 = 0.f;
#define RGNN_GATHER_FETCH_IDX(J)                                                                  \
    _Pragma("unroll") for (int u = 0; u < 4; ++u) {                                               \
        const int jj = min((J) + u, e - 1);                                                       \
        const int k = a.via ? a.via[jj] : jj;                                                     \
        row[u] = a.rowidx ? (a.row_by_k ? a.rowidx[k] : a.rowidx[jj]) : k;                        \
        float cc = a.coef ? a.coef[(size_t)k * a.cstride + head] : 1.f;                           \
        if (a.cabs) cc = fabsf(cc);                                                               \
        c[u] = (J) + u < e ? cc : 0.f;                                                            \
        if (S2) c2[S2 ? u : 0] = (J) + u < e ? a.coef[(size_t)k * a.cstride + a.s2off + head] : 0.f; \
    }
    if (b < e) {
        RGNN_GATHER_FETCH_IDX(b)
    }
    for (int j = b; j < e; j += 4) {
        float v[4][V];
        float cc[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (NT && sizeof(TI) == 4) load_cols_nt(src + (size_t)row[u] * D + cv * V, v[u]);
            else load_cols(src + (size_t)row[u] * D + cv * V, v[u]);
            cc[u] = c[u];
            if (S2) s2 += c2[S2 ? u : 0];
            if (sizeof(TI) == 4 && j + u >= e) zero_cols(v[u]);      // (it may be infinite: no weight 0)
        }
        if (j + 4 < e) {
            RGNN_GATHER_FETCH_IDX(j + 4)
        }
        fma_cols(acc0, cc[0], v[0]);
        fma_cols(acc1, cc[1], v[1]);
        fma_cols(acc0, cc[2], v[2]);
        fma_cols(acc1, cc[3], v[3]);
    }
#undef RGNN_GATHER_FETCH_IDX
    fma_cols(acc0, 1.f, acc1);
    const int slot = a.it.slot[i];
    if (slot < 0) {
        if (R1) add_rank1<D>(a.r1, a.lanes_per_head, (size_t)a.it.row[i], cv, acc0);
        if (EX) add_row<D>(a.extra, (size_t)a.it.row[i], cv, acc0);
        if (S2) add_rank1_own<D>(a.r1, s2, (size_t)a.it.row[i], cv, acc0);
        store_cols(static_cast<TO*>(a.out) + (size_t)a.it.row[i] * D + cv * V, acc0);
        if (S2 && cv % a.lanes_per_head == 0) a.sum2[(size_t)a.it.row[i] * a.sum2_stride + head] = s2;
    } else {
        store_cols(a.partial + (size_t)slot * D + cv * V, acc0);
    }
}

// The whole segments with 2..kShortLen entries, items [first, first + n).  One batch of row loads covers
// such a segment, so the general kernel would spend its time on the item -> indices -> rows -> store
// chain; here a group of lanes takes two of them at a time, all loads of both independent (entries
// past a segment's end repeat its last one with a zero coefficient).
template <int D, typename TI, typename TO, bool R1, bool NT, bool S2 = false, bool EX = false>
__device__ __forceinline__ void gather_short(const GatherArgs& a, int blk, int first, int n) {
    constexpr int V = RowT<TI>::V, LPR = D / V, GPB = 256 / LPR;
    const int g = blk * GPB + threadIdx.x / LPR, cv = threadIdx.x % LPR;
    const int i0 = 2 * g;
    if (i0 >= n) return;
    const TI* __restrict__ src = static_cast<const TI*>(a.src);
    const int head = cv / a.lanes_per_head;
    int b[2], e[2], orow[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int i = first + min(i0 + q, n - 1);
        b[q] = a.it.beg[i];
        e[q] = a.it.end[i];
        orow[q] = a.it.row[i];
    }
    int row[2][kShortLen];
    float c[2][kShortLen], s2[2] = {0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < kShortLen; ++u) {
            const int jj = min(b[q] + u, e[q] - 1);
            const int k = a.via ? a.via[jj] : jj;
            row[q][u] = a.rowidx ? (a.row_by_k ? a.rowidx[k] : a.rowidx[jj]) : k;
            float cc = a.coef ? a.coef[(size_t)k * a.cstride + head] : 1.f;
            if (a.cabs) cc = fabsf(cc);
            c[q][u] = b[q] + u < e[q] ? cc : 0.f;
            if (S2) s2[q] += b[q] + u < e[q] ? a.coef[(size_t)k * a.cstride + a.s2off + head] : 0.f;
        }
    float v[2][kShortLen][V];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < kShortLen; ++u) {
            if (NT && sizeof(TI) == 4) load_cols_nt(src + (size_t)row[q][u] * D + cv * V, v[q][u]);
            else load_cols(src + (size_t)row[q][u] * D + cv * V, v[q][u]);
        }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        float acc[V];
        zero_cols(acc);
#pragma unroll
        for (int u = 0; u < kShortLen; ++u) {
            if (sizeof(TI) == 4 && b[q] + u >= e[q]) zero_cols(v[q][u]);
            fma_cols(acc, c[q][u], v[q][u]);
        }
        if (i0 + q < n) {
            if (R1) add_rank1<D>(a.r1, a.lanes_per_head, (size_t)orow[q], cv, acc);
            if (EX) add_row<D>(a.extra, (size_t)orow[q], cv, acc);
            if (S2) add_rank1_own<D>(a.r1, s2[q], (size_t)orow[q], cv, acc);
            store_cols(static_cast<TO*>(a.out) + (size_t)orow[q] * D + cv * V, acc);
            if (S2 && cv % a.lanes_per_head == 0) a.sum2[(size_t)orow[q] * a.sum2_stride + head] = s2[q];
        }
    }
}

// The whole segments with exactly one entry, items [first, first + n): out[row_i] = c * src[row].
// A group of lanes handles four of them at a time, all loads of the four independent, which keeps
// enough rows in flight where the general kernel would wait on one short dependent chain per item.
template <int D, typename TI, typename TO, bool R1, bool NT, bool EX = false>
__device__ __forceinline__ void gather_single(const GatherArgs& a, int blk, int first, int n) {
    constexpr int V = RowT<TI>::V, LPR = D / V, GPB = 256 / LPR;
    const int g = blk * GPB + threadIdx.x / LPR, cv = threadIdx.x % LPR;
    const int i0 = 4 * g;
    if (i0 >= n) return;
    const TI* __restrict__ src = static_cast<const TI*>(a.src);
    const int head = cv / a.lanes_per_head;
    int j[4], orow[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int i = first + min(i0 + u, n - 1);
        j[u] = a.it.beg[i];
        orow[u] = a.it.row[i];
    }
    int row[4];
    float c[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int k = a.via ? a.via[j[u]] : j[u];
        row[u] = a.rowidx ? (a.row_by_k ? a.rowidx[k] : a.rowidx[j[u]]) : k;
        c[u] = a.coef ? a.coef[(size_t)k * a.cstride + head] : 1.f;
        if (a.cabs) c[u] = fabsf(c[u]);
    }
    float v[4][V];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (NT && sizeof(TI) == 4) load_cols_nt(src + (size_t)row[u] * D + cv * V, v[u]);
        else load_cols(src + (size_t)row[u] * D + cv * V, v[u]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (i0 + u < n) {
#pragma unroll
            for (int q = 0; q < V; ++q) v[u][q] *= c[u];
            if (R1) add_rank1<D>(a.r1, a.lanes_per_head, (size_t)orow[u], cv, v[u]);
            if (EX) add_row<D>(a.extra, (size_t)orow[u], cv, v[u]);
            store_cols(static_cast<TO*>(a.out) + (size_t)orow[u] * D + cv * V, v[u]);
        }
    }
}

// fp32 rows: one launch for the three kinds of items: the first blocks walk the general items (longest
// first), the next ones the 2..kShortLen-entry segments, the last ones the single-entry segments, so the
// short work fills the machine while the long items drain.  bf16 rows: a launch per kind (a lane holds
// twice the columns there, and the registers of the short-segment path would cost the general walk
// its occupancy).
struct GatherRanges { int general_blocks, short_blocks, short_first, short_n, single_first, single_n; };
// R1: the rank-1 term of GatherArgs::r1 is present (fp32 rows only).
template <int D, int ROLE, typename TI, typename TO, bool R1 = false>
__global__ __launch_bounds__(256) void gather_sum_kernel(GatherArgs a, GatherRanges r) {
    const int blk = blockIdx.x;
    if (blk < r.general_blocks) gather_general<D, TI, TO, R1, ROLE == 0, false, ROLE == 3>(a, blk);
    else if (blk < r.general_blocks + r.short_blocks) gather_short<D, TI, TO, R1, ROLE == 0, false, ROLE == 3>(a, blk - r.general_blocks, r.short_first, r.short_n);
    else gather_single<D, TI, TO, R1, ROLE == 0, ROLE == 3>(a, blk - r.general_blocks - r.short_blocks, r.single_first, r.single_n);
}
template <int D, int ROLE, typename TI, typename TO>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(7))) void gather_general_kernel(GatherArgs a) { gather_general<D, TI, TO, false, ROLE == 0>(a, blockIdx.x); }
template <int D, int ROLE, typename TI, typename TO>
__global__ __launch_bounds__(256) void gather_short_kernel(GatherArgs a, int first, int n) { gather_short<D, TI, TO, false, ROLE == 0>(a, blockIdx.x, first, n); }
template <int D, int ROLE, typename TI, typename TO>
__global__ __launch_bounds__(256) void gather_single_kernel(GatherArgs a, int first, int n) { gather_single<D, TI, TO, false, ROLE == 0>(a, blockIdx.x, first, n); }

// NH weighted sums of the same rows in one walk: out[h][row_i] = sum_j coef[k][h] * src[row], k and row as
// in gather_sum_kernel (fp32 rows).  out is [NH][out_rows][D], the partial rows [NH][num_partials][D].
template <int D, int NH>
__device__ __forceinline__ void gather_heads_rows(const GatherArgs& a, int blk, int out_rows, int num_partials) {
    constexpr int LPR = D / 4, IPB = 256 / LPR;
    const int i = blk * IPB + threadIdx.x / LPR, c4 = threadIdx.x % LPR;
    if (i >= a.it.n) return;
    const float* __restrict__ src = static_cast<const float*>(a.src);
    const int b = a.it.beg[i], e = a.it.end[i];
    float4 acc[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) acc[h] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int j = b; j < e; j += 2) {
        float4 x[2];
        float c[2][NH];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int jj = min(j + u, e - 1);
            const int k = a.via ? a.via[jj] : jj;
            const int row = a.rowidx ? (a.row_by_k ? a.rowidx[k] : a.rowidx[jj]) : k;
            x[u] = *reinterpret_cast<const float4*>(src + (size_t)row * D + c4 * 4);
#pragma unroll
            for (int h = 0; h < NH; ++h) c[u][h] = j + u < e ? a.coef[(size_t)k * NH + h] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int h = 0; h < NH; ++h) fma4(acc[h], c[u][h], x[u]);
    }
    const int slot = a.it.slot[i];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        float* o = slot < 0 ? static_cast<float*>(a.out) + ((size_t)h * out_rows + a.it.row[i]) * D
                            : a.partial + ((size_t)h * num_partials + slot) * D;
        *reinterpret_cast<float4*>(o + c4 * 4) = acc[h];
    }
}
template <int D, int NH>
__global__ __launch_bounds__(256) void gather_heads_rows_kernel(GatherArgs a, int out_rows, int num_partials) {
    gather_heads_rows<D, NH>(a, blockIdx.x, out_rows, num_partials);
}

// The two walks of RGAT's backward that need only the edges' (att, dz) and the runs' ds_dst: the first blocks walk the runs by
// relation (U[r][h] = sum_q ds_dst[q][h] X[dst_q], KR columns), the others the pairs with several edges (the gradient rows, D
// columns, and ds_src).  Each is bound by its gathers, and each drains for some microseconds when it is alone: the items of
// the relations are long and few, those of the pairs short and many.  As launches of their own 12.5 and 19 us at 200k edges, so 21;
// 96 and 78 at 2.5M edges and four heads, so 159; 345 and 233 at 10M, so 549.
template <int D, int KR, int NH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void pair_run_walks_kernel(GatherArgs pair, GatherRanges r, GatherArgs run, int run_blocks,
                                                                                                     int out_rows, int num_partials) {
    int blk = blockIdx.x;
    if (blk < run_blocks) {
        if constexpr (NH == 1) gather_general<KR, float, float, false, false>(run, blk);
        else gather_heads_rows<KR, NH>(run, blk, out_rows, num_partials);
        return;
    }
    blk -= run_blocks;
    if (blk < r.general_blocks) gather_general<D, float, float, false, false, true>(pair, blk);
    else gather_short<D, float, float, false, false, true>(pair, blk - r.general_blocks, r.short_first, r.short_n);
}

// out[split_row[s]] = sum of partial rows [split_ptr[s], split_ptr[s+1]).  A workgroup of TH threads owns C4 float4 columns
// (blockIdx.z) of one cut segment (and of one copy of the rows, blockIdx.y): group g of C4 lanes sums partial rows g, g + G,
// g + 2G, ..., four at a time with their loads independent, then the G group sums are added through LDS: in group order,
// or, over more than 32 groups, by halves (a chain of 128 additions raises the error of a relation's sum over its runs
// above that of 64 groups: 3.5e-7 against 3.2e-7 at 1.1M runs, four heads; by halves 3.0e-7 and 8.2 us for 9.6 at 4.3M).  Either way the summation
// order is fixed.
template <int D, typename TO, int TH, int C4>
__global__ __launch_bounds__(TH) void combine_partials_kernel(const int32_t* __restrict__ split_row,
                                                              const int32_t* __restrict__ split_ptr,
                                                              const float* __restrict__ partial, TO* __restrict__ out,
                                                              size_t partial_copy, size_t out_copy, Rank1 r1, int lanes_per_head, const float* extra) {
    constexpr int G = TH / C4;
    __shared__ float4 red[TH];
    partial += blockIdx.y * partial_copy;
    out += blockIdx.y * out_copy;
    const int s = blockIdx.x, g = threadIdx.x / C4, c = threadIdx.x % C4, c4 = blockIdx.z * C4 + c;
    const int p0 = split_ptr[s], p1 = split_ptr[s + 1];
    float4 acc0 = make_float4(0.f, 0.f, 0.f, 0.f), acc1 = acc0;
    for (int p = p0 + g; p < p1; p += 4 * G) {
        float4 r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) r[u] = *reinterpret_cast<const float4*>(partial + (size_t)min(p + u * G, p1 - 1) * D + c4 * 4);
        fma4(acc0, 1.f, r[0]);
        if (p + G < p1) fma4(acc1, 1.f, r[1]);
        if (p + 2 * G < p1) fma4(acc0, 1.f, r[2]);
        if (p + 3 * G < p1) fma4(acc1, 1.f, r[3]);
    }
    fma4(acc0, 1.f, acc1);
    red[threadIdx.x] = acc0;
    __syncthreads();
    constexpr bool tree = G > 32;
    if (tree) {
#pragma unroll
        for (int h = G / 2; h > 0; h /= 2) {
            if (g < h) fma4(red[threadIdx.x], 1.f, red[threadIdx.x + h * C4]);
            __syncthreads();
        }
    }
    if (g == 0) {
        float4 t = red[c];
        if (!tree) {
            const int n = min(G, p1 - p0);        // groups that had a piece
            for (int k = 1; k < n; ++k) fma4(t, 1.f, red[k * C4 + c]);
        }
        float tv[4] = {t.x, t.y, t.z, t.w};
        add_rank1<D>(r1, lanes_per_head, (size_t)split_row[s], c4, tv);
        add_row<D>(extra, (size_t)split_row[s], c4, tv);
        store_cols(out + (size_t)split_row[s] * D + c4 * 4, tv);
    }
}
// Hub nodes and pairs: mostly two or three pieces per cut segment and thousands of segments, so small workgroups (1024
// threads with two loads in flight took 33 us for the destinations of a graph of 2M edges at width 128, 256 threads with
// four 11 us).  Run lists of relations: a few dozen segments with thousands of pieces, so large workgroups on narrow
// column ranges (843k runs of 60 relations in 13k pieces, width 128: 256 threads 61 us, 1024 on whole rows 26 us, on 8
// float4 13 us).
inline bool few_long_segments(const ItemList& L) { return L.num_partials > 32 * L.num_split; }

// Cut destinations of a softmax-weighted sum: the pieces carry (max m_i, sum s_i of exp(l - m_i)) per head and the
// unnormalised row; out[v] = sum_i exp(m_i - M) partial_i / S with M = max_i m_i, S = sum_i s_i exp(m_i - M).  One workgroup
// per cut destination: group g of D/4 lanes takes the pieces g, g + G, ... four at a time (their loads independent) in the
// running-maximum form, and the G group results are merged in group order through LDS.  H heads are equal column slices.
// The rows carry pow2_share(piece_len) and get pow2_share(number of pieces) here, so that a sum whose mean fits in fp32 does too.
// FULL: expf (HGT, like its walks), otherwise __expf (RGAT, like its walks; expf adds 1 us at 300k nodes).
template <int D, int H, typename TO, bool FULL>
__global__ __launch_bounds__(256) void combine_softmax_kernel(const int32_t* __restrict__ split_row,
                                                              const int32_t* __restrict__ split_ptr,
                                                              const float* __restrict__ partial,
                                                              const float2* __restrict__ part_ms, TO* __restrict__ out,
                                                              float2* __restrict__ ms, const int32_t* __restrict__ ms_row, int piece_len) {
    constexpr int LPR = D / 4, G = 256 / LPR, LPH = LPR / H;
    auto ex = [](float x) { return FULL ? expf(x) : __expf(x); };
    __shared__ float4 red[256];
    __shared__ float2 redms[G][H];
    const int s = blockIdx.x, g = threadIdx.x / LPR, c = threadIdx.x % LPR, head = c / LPH;
    const int p0 = split_ptr[s], p1 = split_ptr[s + 1];
    const float share = pow2_share(p1 - p0);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float M = -INFINITY, S = 0.f;
    for (int p = p0 + g; p < p1; p += 4 * G) {
        float2 t[4];
        float4 r[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int pp = min(p + u * G, p1 - 1);
            t[u] = part_ms[(size_t)pp * H + head];
            r[u] = *reinterpret_cast<const float4*>(partial + (size_t)pp * D + c * 4);
        }
        float mn = M;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (p + u * G >= p1) {                // the repeated piece counts as nothing (it may be infinite: no weight 0)
                t[u] = make_float2(-INFINITY, 0.f);
                r[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
            mn = fmaxf(mn, t[u].x);
        }
        const float base = softmax_base(mn), sc = ex(M - base);       // 0 for the first four pieces
        S *= sc;
        acc.x *= sc; acc.y *= sc; acc.z *= sc; acc.w *= sc;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float w = ex(t[u].x - base);
            S += w * t[u].y;
            fma4(acc, w * share, r[u]);
        }
        M = mn;
    }
    red[threadIdx.x] = acc;
    if (c % LPH == 0) redms[g][head] = make_float2(M, S);
    __syncthreads();
    if (g == 0) {
        const int n = min(G, p1 - p0);            // groups that had a piece
        for (int k = 1; k < n; ++k) M = fmaxf(M, redms[k][head].x);
        S = 0.f;
        float t[4] = {0.f, 0.f, 0.f, 0.f};
        for (int k = 0; k < n; ++k) {
            const float2 q = redms[k][head];
            const float w = ex(q.x - softmax_base(M));
            const float4 r = red[k * LPR + c];
            S += w * q.y;
            t[0] += w * r.x; t[1] += w * r.y; t[2] += w * r.z; t[3] += w * r.w;
        }
        // (ms_row: the runs of RGAT, of which one without weight gets the zero row)
        const float inv = ms_row && S == 0.f ? 0.f : 1.f / S * (1.f / share) * (1.f / pow2_share(piece_len));
        const size_t v = (size_t)split_row[s];
#pragma unroll
        for (int q = 0; q < 4; ++q) t[q] *= inv;
        store_cols(out + v * D + c * 4, t);
        if (c % LPH == 0) ms[(ms_row ? (size_t)ms_row[v] : v) * H + head] = make_float2(M, S);
    }
}

// ------------------------------------------------------------------ edge-parallel aggregation (comparison schedule)

// out[dst_e] += |att_e| * Hs[pair_e] over equal shares of the CSR edge list: a lane group takes
// kEdgeChunk consecutive edges, sums in registers while the destination stays the same and adds the sum
// to the output row with atomic adds when it changes (the thesis' traversal template: partial
// aggregation in the thread, then atomicAdd to global memory).  Work is balanced by construction (no
// work lists), the price is the atomics.  out must be zero on entry.  The destination of a CSR edge is
// run_dst[in_run[e]].
constexpr int kEdgeChunk = 16;
template <int D>
__global__ __launch_bounds__(256) void aggregate_edge_parallel_kernel(int64_t E, const int32_t* __restrict__ in_pair,
                                                                      const int32_t* __restrict__ in_run,
                                                                      const int32_t* __restrict__ run_dst,
                                                                      const float* __restrict__ att,
                                                                      const float* __restrict__ Hs, float* __restrict__ out) {
    constexpr int LPR = D / 4, GPB = 256 / LPR;
    const int64_t e0 = ((int64_t)blockIdx.x * GPB + threadIdx.x / LPR) * kEdgeChunk;
    const int c4 = threadIdx.x % LPR;
    if (e0 >= E) return;
    const int64_t e1 = e0 + kEdgeChunk < E ? e0 + kEdgeChunk : E;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    int cur = run_dst[in_run[e0]];
    auto flush = [&](int v) {
        // the hardware's fp32 add on memory (no compare-and-swap loop); ordinary device memory
        float* o = out + (size_t)v * D + c4 * 4;
        unsafeAtomicAdd(o + 0, acc.x);
        unsafeAtomicAdd(o + 1, acc.y);
        unsafeAtomicAdd(o + 2, acc.z);
        unsafeAtomicAdd(o + 3, acc.w);
    };
    for (int64_t e = e0; e < e1; ++e) {
        const int v = run_dst[in_run[e]];
        if (v != cur) {
            flush(cur);
            acc = make_float4(0.f, 0.f, 0.f, 0.f);
            cur = v;
        }
        fma4(acc, fabsf(att[e]), *reinterpret_cast<const float4*>(Hs + (size_t)in_pair[e] * D + c4 * 4));
    }
    flush(cur);
}
__global__ void zero_f32_kernel(size_t n, float* __restrict__ x) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = 0.f;
}

// ------------------------------------------------------------------ sums of the weight gradients' shares

// dW[s] (and Avec[s]) = sum of the partial slots of segment s; kn / kd = floats of a slot's matrix / vector part, both
// multiples of 4.  A workgroup owns C4 consecutive float4 of one segment's slots; its G lane groups take the slots in turn,
// four loads in flight each, and the group sums are added in four chains through LDS, so the result does not depend on
// scheduling (as one chain the error of a self-loop's dW at 120k nodes was 1.47e-7, now 1.27e-7).  Bound by the chain of loads of the
// segment with the most slots, and with thousands of segments by their workgroups' start.
__device__ __forceinline__ void store_slot_sum(const ShareSums::Job& j, int seg, int i, float4 t) {
    if (i < j.kn) *reinterpret_cast<float4*>(j.dW + (size_t)seg * j.kn + i) = t;
    else *reinterpret_cast<float4*>(j.dW2 + (size_t)seg * j.kd + (i - j.kn)) = t;
}
template <int G, int C4>
__device__ __forceinline__ void slot_sum_groups(const ShareSums::Job& j, int seg, int col_blk, float4* red) {
    const int c = threadIdx.x % C4, g = threadIdx.x / C4;
    const int i = (col_blk * C4 + c) * 4, slot_sz = j.kn + j.kd;
    const bool on = i < j.used;
    float4 s0 = make_float4(0.f, 0.f, 0.f, 0.f), s1 = s0;
    const int b = j.seg_slot_ptr[seg], e = j.seg_slot_ptr[seg + 1];
    if (on) {
        const float* p = j.part + i;
        int sl = b + g;
        for (; sl + 3 * G < e; sl += 4 * G) {
            const float4 x0 = *reinterpret_cast<const float4*>(p + (size_t)sl * slot_sz);
            const float4 x1 = *reinterpret_cast<const float4*>(p + (size_t)(sl + G) * slot_sz);
            const float4 x2 = *reinterpret_cast<const float4*>(p + (size_t)(sl + 2 * G) * slot_sz);
            const float4 x3 = *reinterpret_cast<const float4*>(p + (size_t)(sl + 3 * G) * slot_sz);
            s0.x += x0.x + x2.x; s0.y += x0.y + x2.y; s0.z += x0.z + x2.z; s0.w += x0.w + x2.w;
            s1.x += x1.x + x3.x; s1.y += x1.y + x3.y; s1.z += x1.z + x3.z; s1.w += x1.w + x3.w;
        }
        for (; sl < e; sl += G) {
            const float4 x0 = *reinterpret_cast<const float4*>(p + (size_t)sl * slot_sz);
            s0.x += x0.x; s0.y += x0.y; s0.z += x0.z; s0.w += x0.w;
        }
    }
    red[g * C4 + c] = make_float4(s0.x + s1.x, s0.y + s1.y, s0.z + s1.z, s0.w + s1.w);
    __syncthreads();
    constexpr int CH = C4 < 64 ? 64 / C4 : 1;              // chains over the groups, one wavefront's worth of lanes
    if (g >= CH) return;
    float4 t = red[g * C4 + c];
#pragma unroll
    for (int k = g + CH; k < G; k += CH) {
        const float4 x = red[k * C4 + c];
        t.x += x.x; t.y += x.y; t.z += x.z; t.w += x.w;
    }
#pragma unroll
    for (int o = C4; o < CH * C4; o <<= 1) {
        t.x += __shfl_xor(t.x, o); t.y += __shfl_xor(t.y, o); t.z += __shfl_xor(t.z, o); t.w += __shfl_xor(t.w, o);
    }
    if (g == 0 && on) store_slot_sum(j, seg, i, t);
}
// Many segments of a few slots each: a lane per float4 of the slot, eight slots in flight, added in four chains; bound by the slots'
// bytes.  (In blocks as above with G = 4 it was bound by the workgroups' start: 2000 segments of width 64 in one or two slots each 24 us,
// so 14; 500 of width 128 in bf16 25, so 17; HGT's 300 folded pairs of weights 54, so 36.  With 16 slots in flight the kernel's
// registers halve the wavefronts of the other blocks: 42 us for 31 with 30 relations in bf16.)
__device__ __forceinline__ void slot_sum_few(const ShareSums::Job& j, int seg, int col_blk) {
    const unsigned i = (col_blk * 256u + threadIdx.x) * 4;
    const size_t slot_sz = j.kn + j.kd;
    if ((int)i >= j.used) return;
    int sl = j.seg_slot_ptr[seg];
    const int e = j.seg_slot_ptr[seg + 1];
    auto load = [&](int slot) { return *reinterpret_cast<const float4*>(j.part + slot * slot_sz + i); };
    float4 s[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (; sl + 8 <= e; sl += 8) {
        float4 x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = load(sl + k);
#pragma unroll
        for (int k = 0; k < 8; ++k) fma4(s[k & 3], 1.f, x[k]);
    }
    for (; sl < e; sl += 4) {
        float4 x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = sl + k < e ? load(sl + k) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int k = 0; k < 4; ++k) fma4(s[k], 1.f, x[k]);
    }
    fma4(s[0], 1.f, s[1]);
    fma4(s[2], 1.f, s[3]);
    fma4(s[0], 1.f, s[2]);
    store_slot_sum(j, seg, (int)i, s[0]);
}

// The other kind of shares that RGAT's backward leaves per relation: U[h][r] from the pieces of r's run list (SumArgs: one copy of
// rows per head).  Independent of the slots, so one launch sums both.  A workgroup takes 16 columns of one relation and head,
// 64 lane groups take its pieces in turn in four chains, and the group sums are added by halves.  Bound by
// the chain of loads of the largest relation (4.3M runs of 200 relations, 17k pieces, width 64: both sums 17 us, as launches of
// their own 7 and 8.5; at 93k runs of 50 relations 6 us, two launches of 6).
__device__ __forceinline__ void piece_sum_block(const SumArgs& u, int blk, float4* red) {
    constexpr int C4 = 4, G = 64;
    const int cols = u.D / (4 * C4), s = blk / (cols * u.copies), h = blk / cols % u.copies;
    const int c = threadIdx.x % C4, g = threadIdx.x / C4, c4 = blk % cols * C4 + c;
    const float* __restrict__ p = u.partial + (size_t)h * u.partial_copy + c4 * 4;
    const int p0 = u.split_ptr[s], p1 = u.split_ptr[s + 1];
    float4 acc[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) acc[x] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k = p0 + g; k < p1; k += 4 * G) {
        float4 r[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) r[x] = *reinterpret_cast<const float4*>(p + (size_t)min(k + x * G, p1 - 1) * u.D);
#pragma unroll
        for (int x = 0; x < 4; ++x)
            if (k + x * G < p1) fma4(acc[x], 1.f, r[x]);
    }
    fma4(acc[0], 1.f, acc[1]);
    fma4(acc[2], 1.f, acc[3]);
    fma4(acc[0], 1.f, acc[2]);
    red[threadIdx.x] = acc[0];
    __syncthreads();
#pragma unroll
    for (int o = G / 2; o > 0; o /= 2) {
        if (g < o) fma4(red[threadIdx.x], 1.f, red[threadIdx.x + o * C4]);
        __syncthreads();
    }
    if (g == 0) *reinterpret_cast<float4*>(u.out + (size_t)h * u.out_copy + (size_t)u.split_row[s] * u.D + c4 * 4) = red[c];
}
// One launch for all shares of a backward pass, a list's blocks of any kind one after the other.  Above eight slots per segment (a
// self-loop weight, node types, few relations) many lane groups on narrow column ranges win.  Below, a lane alone on its slots, unless
// the segment with the most slots would take it longer than the list's bytes take (frequencies of Zipf 1.2, 500 relations, 1.2M edges:
// width 32 9.9 us, in four groups 7; width 64 11.9 and 10.7; in bf16 at width 128, where the bytes take longer, 20 and 30).  HGT
// in bf16, three lists: 54 us as three launches, now 38 (2M nodes, 5.4M pairs), 38 and 31 (200k nodes); in fp32 at 300k edges four
// launches of 6, now one of 7; RGCN with a self-loop 13 and 7.  (With workgroups of 512 threads 59 and 39 us in the first two.  N is
// a template parameter so that the jobs' fields are loaded together.)
template <int N>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(7))) void sum_shares_kernel(ShareSums s) {
    __shared__ float4 red[256];
    int blk = flat_block();
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const ShareSums::Job j = s.job[k];
        if (blk < j.blocks) {
            const int seg = blk / j.col_blocks, cb = blk % j.col_blocks;
            if (j.kind == ShareSums::kMany) slot_sum_groups<16, 16>(j, seg, cb, red);
            else if (j.kind == ShareSums::kUneven) slot_sum_groups<4, 64>(j, seg, cb, red);
            else slot_sum_few(j, seg, cb);
            return;
        }
        blk -= j.blocks;
    }
    if (blk < s.pieces.blocks()) {
        piece_sum_block(s.pieces, blk, red);
        return;
    }
    blk -= (int)s.pieces.blocks();
    if (blk < s.pieces2.blocks()) piece_sum_block(s.pieces2, blk, red);
}

rgnn_status_t ShareSums::add(const TileList& tiles, const float* part, int kn, int kd, float* dW, float* dW2) {
    if (n == kMax) RGNN_FAIL(RGNN_EUNSUPPORTED, "weight-gradient sums: more than %d lists", kMax);
    const int used = dW2 ? kn + kd : kn;
    const int kind = tiles.num_slots > 8 * tiles.num_segs ? kMany : (int64_t)tiles.max_seg_slots << 16 > (int64_t)tiles.num_slots * used ? kUneven : kFew;
    const int floats = kind == kMany ? 64 : kind == kUneven ? 256 : 1024, cols = (used + floats - 1) / floats;
    if ((int64_t)tiles.num_segs * cols > INT32_MAX / (kMax + 1)) RGNN_FAIL(RGNN_EUNSUPPORTED, "weight-gradient sums: %d segments are too many", tiles.num_segs);
    job[n++] = Job{part, tiles.seg_slot_ptr, tiles.num_segs * cols, cols, kind, kn, kd, used, dW, dW2};
    return RGNN_OK;
}
rgnn_status_t ShareSums::launch(hipStream_t st) {
    int64_t blocks = pieces.blocks() + pieces2.blocks();
    for (int k = 0; k < n; ++k) blocks += job[k].blocks;
    if (blocks > INT32_MAX / 2) RGNN_FAIL(RGNN_EUNSUPPORTED, "weight-gradient sums: too many segments");
    if (blocks > 0) {
        KernelTimer kt(st, "typed_linear_bwd.reduce");
        auto kern = n == 1 ? sum_shares_kernel<1> : n == 2 ? sum_shares_kernel<2> : n == 3 ? sum_shares_kernel<3> : sum_shares_kernel<4>;
        hipLaunchKernelGGL(kern, flat_grid(blocks), dim3(256), 0, st, *this);
        RGNN_CHECK_LAUNCH();
    }
    n = 0;
    pieces = pieces2 = SumArgs{};
    return RGNN_OK;
}
rgnn_status_t typed_linear_slot_reduce(const TileList& tiles, const float* part, int kn, int kd, float* dW, float* dW2, hipStream_t st,
                                       ShareSums* sums) {
    ShareSums own;
    RGNN_TRY((sums ? sums : &own)->add(tiles, part, kn, kd, dW, dW2));
    return sums ? RGNN_OK : own.launch(st);
}

// ------------------------------------------------------------------ RGAT parameter-gradient epilogue

// Per relation r, with A[r][h] = sum_p ds_src[p][h] X[src_p], U[h][r] = sum_q ds_dst[q][h] X[dst_q] and h(n) the head of column n:
//   dw_s[r][n] = sum_k A[r][h(n)][k] W[r][k][n] (without A the caller forms dw_s from the message rows),
//   dw_t[r][n] = sum_k U[h(n)][r][k] W[r][k][n],
//   dW[r][k][n] += U[h(n)][r][k] w_t[r][n], and with one head + A[r][k] w_s[r][n] (with several, the rows that dW came from hold it).
// Blocks (r, j < nd / 32) form 32 columns of the two vectors each (the eight lanes of a column take the k index in turn and are
// added in order through LDS); blocks (r, nd / 32 + j) update 1024 consecutive elements of dW[r] each, four per lane (a lane's four
// columns are one head's).  nd is a power of two, at least 32.  (With all columns of a relation in one workgroup, 31 us for 60
// relations of width 128 and one head, 38 for 101 of width 64 and four; so, 6 and 8.)
__device__ __forceinline__ void param_finish_block(const RgatFinish& f, int blk, float* red) {
    const int per_rel = f.nd / 32 + (f.kd * f.nd + 1023) / 1024, r = blk / per_rel, y = blk % per_rel;
    const int tid = threadIdx.x, kd = f.kd, nd = f.nd, ln = 31 - __clz(nd), ld = ln - (31 - __clz(f.H));     // log2 of a head's width
    const float* Wr = f.W + (size_t)r * kd * nd;
    if (y < nd / 32) {
        const int n = y * 32 + (tid & 31), ks = tid >> 5, h = n >> ld;
        const float* Ur = f.U + ((size_t)h * f.R + r) * kd;
        const float* Ar = f.A + ((size_t)r * f.H + h) * kd;
        float s = 0.f, t = 0.f;
#pragma unroll 8
        for (int k = ks; k < kd; k += 8) {
            const float w = Wr[k * nd + n];
            t += Ur[k] * w;
            if (f.A) s += Ar[k] * w;
        }
        red[tid] = s;
        red[256 + tid] = t;
        __syncthreads();
        if (ks == 0) {
            for (int q = 1; q < 8; ++q) {
                s += red[q * 32 + tid];
                t += red[256 + q * 32 + tid];
            }
            if (f.A) f.dw_s[(size_t)r * nd + n] = s;
            f.dw_t[(size_t)r * nd + n] = t;
        }
        return;
    }
    const int i = ((y - nd / 32) * 256 + tid) * 4;
    if (i >= kd * nd) return;
    const int k = i >> ln, n = i & (nd - 1);
    const float u = f.U[((size_t)(n >> ld) * f.R + r) * kd + k];
    const float4 wt = *reinterpret_cast<const float4*>(f.w_t + (size_t)r * nd + n);
    float4* o = reinterpret_cast<float4*>(f.dW + (size_t)r * kd * nd + i);
    float4 v = *o;
    if (f.H == 1) {
        const float a = f.A[(size_t)r * kd + k];
        const float4 ws = *reinterpret_cast<const float4*>(f.w_s + (size_t)r * nd + n);
        v.x += a * ws.x + u * wt.x;
        v.y += a * ws.y + u * wt.y;
        v.z += a * ws.z + u * wt.z;
        v.w += a * ws.w + u * wt.w;
    } else {
        v.x += u * wt.x;
        v.y += u * wt.y;
        v.z += u * wt.z;
        v.w += u * wt.w;
    }
    *o = v;
}

// ------------------------------------------------------------------ dX assembly

// dX[u] = sum_{p in srcpair(u)} dXp[p]  +  sum_{q in runs(u)} sum_h ds_dst[q][h] * wtp[run_rel[q]][h]  +  extra[u]
// (second and third terms optional).
struct NodeSumArgs {
    Items it;             // pairs by source node, ordered by length, never cut
    const int32_t* srcpair_idx;
    const void* dXp;      // rows of TI
    const void* dXp2;     // a second tensor of per-pair rows, summed with the first
    const int32_t* dst_run_ptr;
    const int32_t* run_rel;
    const float* ds_dst;  // [Q][H]
    const float* wtp;     // [R][H][D]
    const float* extra;
    void* dX;             // rows of TO
};

// RB runs of the run term, H heads each: their relations and coefficients (entries past the end repeat the last one with zero
// coefficients), and the H folded vectors of each relation.
template <int D, int V, int H, int RB>
struct RunBatch {
    struct __align__(4 * H) Coef { float v[H]; };
    int rel[RB];
    float c[RB][H];
    __device__ __forceinline__ void fetch(const NodeSumArgs& a, int q, int qe) {
#pragma unroll
        for (int t = 0; t < RB; ++t) {
            const int x = min(q + t, qe - 1);
            rel[t] = a.run_rel[x];
            const Coef k = *reinterpret_cast<const Coef*>(a.ds_dst + (size_t)x * H);
#pragma unroll
            for (int h = 0; h < H; ++h) c[t][h] = q + t < qe ? k.v[h] : 0.f;
        }
    }
    __device__ __forceinline__ void rows(const NodeSumArgs& a, int cv, float (&w)[RB * H][V]) const {
#pragma unroll
        for (int t = 0; t < RB; ++t)
#pragma unroll
            for (int h = 0; h < H; ++h) load_cols(a.wtp + ((size_t)rel[t] * H + h) * D + cv * V, w[t * H + h]);
    }
    __device__ __forceinline__ void add(const float (&w)[RB * H][V], float (&acc)[V], float (&acc1)[V]) const {
#pragma unroll
        for (int x = 0; x < RB * H; ++x) fma_cols(x & 1 ? acc1 : acc, c[x / H][x % H], w[x]);
    }
    // the runs q, q + step, ... in batches, relations and coefficients one batch ahead of the rows
    __device__ __forceinline__ void walk(const NodeSumArgs& a, int q, int qe, int step, int cv, float (&acc)[V], float (&acc1)[V]) {
        if (q >= qe) return;
        fetch(a, q, qe);
        for (; q < qe; q += step) {
            float w[RB * H][V], cq[RB][H];
            rows(a, cv, w);
#pragma unroll
            for (int t = 0; t < RB; ++t)
#pragma unroll
                for (int h = 0; h < H; ++h) cq[t][h] = c[t][h];
            if (q + step < qe) fetch(a, q + step, qe);
#pragma unroll
            for (int x = 0; x < RB * H; ++x) fma_cols(x & 1 ? acc1 : acc, cq[x / H][x % H], w[x]);
        }
    }
};

// H > 0: the destination-run term is present, with H heads (RGAT); H = 0: the kernel only sums pair rows; TWO: pair rows of
// two tensors (HGT: the key and the message halves of the input gradient).
//
// A lane group per node.  A popular destination has a run of every relation: its run term is shared by all lane groups of its
// wavefront, and a run costs one relation and one load for the coefficients of all heads.  (With a lane group alone on it and an
// entry with loads of its own per (run, head), 250k nodes, 1.1M runs of 101 relations and four heads took 234 us, now 178; with one
// head, 1M nodes and 4.3M runs of 200 relations 519 us, now 504.)  With the run term, the first `fin.blocks` blocks finish the
// layer's parameter gradients, which nothing here reads.
template <int D, typename TI, typename TO, int H, bool TWO>
__global__ __launch_bounds__(256) void node_grad_sum_kernel(NodeSumArgs a, RgatFinish fin) {
    constexpr bool RUNS = H > 0;
    __shared__ float red[RUNS ? 512 : 1];
    const int blk = flat_block();
    if (RUNS && blk < fin.blocks) {
        param_finish_block(fin, blk, red);
        return;
    }
    constexpr int V = RowT<TI>::V, LPR = D / V, IPB = 256 / LPR, G = 64 / LPR;
    constexpr int HH = RUNS ? H : 1, RB = HH == 1 ? 4 : HH <= 4 ? 2 : 1;     // runs per batch
    constexpr int ALONE = 8 * RB;                                           // runs that a lane group walks by itself
    static_assert(!RUNS || (sizeof(TI) == 4 && !TWO), "the run term goes with fp32 rows of one tensor");
    const int i0 = (blk - (RUNS ? fin.blocks : 0)) * IPB + threadIdx.x / LPR, cv = threadIdx.x % LPR;
    const bool on = i0 < a.it.n;
    if (RUNS ? !__any(on) : !on) return;            // (with runs, the lanes past the end help with other nodes')
    const int i = min(i0, a.it.n - 1);
    const TI* __restrict__ dXp = static_cast<const TI*>(a.dXp);
    const TI* __restrict__ dXp2 = static_cast<const TI*>(a.dXp2);
    const int u = a.it.row[i];
    const int b = a.it.beg[i], e = on ? a.it.end[i] : b;
    int qb = 0, qe = 0;
    if (RUNS) {
        qb = a.dst_run_ptr[u];
        qe = on ? a.dst_run_ptr[u + 1] : qb;
    }
    float acc[V], acc1[V];
    zero_cols(acc);
    zero_cols(acc1);
    // The first four pairs and the first runs of the node are fetched together (a node has
    // about as many of either as one batch holds), so their two index -> row chains overlap.
    int pi[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) pi[t] = b + t < e ? a.srcpair_idx[b + t] : -1;
    RunBatch<D, V, HH, RB> first;
    const bool runs = RUNS && qb < qe;
    if (runs) first.fetch(a, qb, qe);
    if (a.extra && on) load_cols(a.extra + (size_t)u * D + cv * V, acc);
    {
        float v[4][V], w[4][V], rw[RB * HH][V];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (pi[t] >= 0) load_cols_nt(dXp + (size_t)pi[t] * D + cv * V, v[t]);
            else zero_cols(v[t]);
            if (TWO && pi[t] >= 0) load_cols(dXp2 + (size_t)pi[t] * D + cv * V, w[t]);
            else zero_cols(w[t]);
        }
        if (runs) first.rows(a, cv, rw);
        fma_cols(acc, 1.f, v[0]);
        fma_cols(acc1, 1.f, v[1]);
        fma_cols(acc, 1.f, v[2]);
        fma_cols(acc1, 1.f, v[3]);
        if (TWO) {
            fma_cols(acc, 1.f, w[0]);
            fma_cols(acc1, 1.f, w[1]);
            fma_cols(acc, 1.f, w[2]);
            fma_cols(acc1, 1.f, w[3]);
        }
        if (runs) first.add(rw, acc, acc1);
    }
    for (int j = b + 4; j < e; j += 4) {
        float v[4][V], w[4][V];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            zero_cols(v[t]);
            zero_cols(w[t]);
            if (j + t < e) {
                const size_t p = (size_t)a.srcpair_idx[j + t];
                load_cols_nt(dXp + p * D + cv * V, v[t]);
                if (TWO) load_cols(dXp2 + p * D + cv * V, w[t]);
            }
        }
        fma_cols(acc, 1.f, v[0]);
        fma_cols(acc1, 1.f, v[1]);
        fma_cols(acc, 1.f, v[2]);
        fma_cols(acc1, 1.f, v[3]);
        if (TWO) {
            fma_cols(acc, 1.f, w[0]);
            fma_cols(acc1, 1.f, w[1]);
            fma_cols(acc, 1.f, w[2]);
            fma_cols(acc1, 1.f, w[3]);
        }
    }
    if (RUNS) {
        const int left = qe - (qb + RB), sub = (threadIdx.x & 63) / LPR;
        if (left > 0 && left <= ALONE) first.walk(a, qb + RB, qe, RB, cv, acc, acc1);
        if (__ballot(left > ALONE)) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int from = __builtin_amdgcn_readlane(qb, g * LPR) + RB, to = __builtin_amdgcn_readlane(qe, g * LPR);
                if (to - from <= ALONE) continue;
                float s0[V], s1[V];
                zero_cols(s0);
                zero_cols(s1);
                first.walk(a, from + sub * RB, to, G * RB, cv, s0, s1);
                fma_cols(s0, 1.f, s1);
#pragma unroll
                for (int o = LPR; o < 64; o <<= 1)
#pragma unroll
                    for (int q = 0; q < V; ++q) s0[q] += __shfl_xor(s0[q], o);
                if (sub == g) fma_cols(acc, 1.f, s0);
            }
        }
    }
    if (RUNS && !on) return;
    fma_cols(acc, 1.f, acc1);
    store_cols(static_cast<TO*>(a.dX) + (size_t)u * D + cv * V, acc);
}

// ------------------------------------------------------------------ elementwise

// Rows per run: dX[v] += sum over v's runs of ds_dst[q] wtp[run_rel[q]].  A group of D / 4 lanes per destination, relations and coefficients of
// D / 4 runs at a time, a lane each; wtp in LDS where it fits (persistent workgroups).  The first `fin.blocks` workgroups finish the
// layer's parameter gradients.  Bound by the rows of dX, read and written: 900k destinations of width 64, 4.4M runs 252 us with a load of the
// folded vector per run, 123 with it in LDS, 117 by length.
constexpr int kRunTermThreads = 512;
template <int D, bool LDSW>
__global__ __launch_bounds__(kRunTermThreads) void run_term_kernel(Items it, int R, const int32_t* __restrict__ dst_run_ptr, const int32_t* __restrict__ run_rel,
                                                                   const float* __restrict__ ds_dst, const float* __restrict__ wtp, float* __restrict__ dX,
                                                                   RgatFinish fin) {
    constexpr int LPR = D / 4, GPB = kRunTermThreads / LPR;
    extern __shared__ __align__(16) float smem[];          // max(R * D, 512) floats
    if ((int)blockIdx.x < fin.blocks) {
        if (threadIdx.x >= 256) return;                    // (whole wavefronts, which the barriers inside no longer count)
        param_finish_block(fin, blockIdx.x, smem);
        return;
    }
    const float* w = wtp;
    if (LDSW) {
        for (int i = threadIdx.x; i < R * D / 4; i += kRunTermThreads) reinterpret_cast<float4*>(smem)[i] = reinterpret_cast<const float4*>(wtp)[i];
        __syncthreads();
        w = smem;
    }
    // The next item's first runs and its row are asked for before this one's sums, and the ends of the one after it.  The items lie by
    // length, so that those of a wavefront end together; the first piece of a cut destination takes the whole of it.
    const int c = threadIdx.x % LPR, step = (gridDim.x - fin.blocks) * GPB, last = it.n - 1;
    int i = (blockIdx.x - fin.blocks) * GPB + threadIdx.x / LPR;
    if (i >= it.n) return;
    int b = it.beg[i], e = it.end[i], v = it.row[i], cut = it.slot[i];
    int k1 = min(i + step, last), bn = it.beg[k1], en = it.end[k1], vn = it.row[k1], cutn = it.slot[k1];
    int j = max(min(b + c, e - 1), 0), rel = run_rel[j];
    float ds = ds_dst[j];
    float4 x = *reinterpret_cast<const float4*>(dX + (size_t)v * D + c * 4);
    for (; i < it.n; i += step) {
        j = max(min(bn + c, en - 1), 0);
        const int reln = run_rel[j];
        const float dsn = ds_dst[j];
        const float4 xn = *reinterpret_cast<const float4*>(dX + (size_t)vn * D + c * 4);
        k1 = min(i + 2 * step, last);
        const int bnn = it.beg[k1], enn = it.end[k1], vnn = it.row[k1], cutnn = it.slot[k1];
        if (cut >= 0) e = b == dst_run_ptr[v] ? dst_run_ptr[v + 1] : b;
        float4 acc1 = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int jc = b; jc < e; jc += LPR) {
            if (jc > b) {
                j = min(jc + c, e - 1);
                rel = run_rel[j];
                ds = ds_dst[j];
            }
            const int n = min(LPR, e - jc);
            const float d = c < n ? ds : 0.f;
#pragma unroll
            for (int k = 0; k < LPR; k += 2) {
                if (k >= n) break;
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    fma4(t ? acc1 : x, group_lane<LPR>(d, k + t), *reinterpret_cast<const float4*>(w + (size_t)group_lane<LPR>(rel, k + t) * D + c * 4));
            }
        }
        fma4(x, 1.f, acc1);
        if (b < e) *reinterpret_cast<float4*>(dX + (size_t)v * D + c * 4) = x;
        b = bn; e = en; v = vn; cut = cutn; bn = bnn; en = enn; vn = vnn; cutn = cutnn; rel = reln; ds = dsn; x = xn;
    }
}

__global__ void relu_kernel(size_t n, float* __restrict__ x) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = x[i] > 0.f ? x[i] : 0.f;
}
// y = (ref > 0) ? g : 0 on fp32 or bf16 storage (G: float or uint16_t); `ref` is the fp32 layer output.  BOTH (bf16): the
// masked gradient also in fp32, for the self-loop kernels.  V elements per thread.  Bound by its bytes: at 120k nodes of
// width 64 one element per thread took 26.6 us, 17.9.
template <typename G, bool BOTH, int V>
__global__ __launch_bounds__(256) void relu_grad_kernel(size_t n, const float* __restrict__ ref, const G* __restrict__ g,
                                                        G* __restrict__ y, float* __restrict__ y32) {
    typedef float vf __attribute__((ext_vector_type(V)));
    typedef G vg __attribute__((ext_vector_type(V)));
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * V;
    if (i >= n) return;
    const vf r = *reinterpret_cast<const vf*>(ref + i);
    vg t = *reinterpret_cast<const vg*>(g + i);
    vf w;
#pragma unroll
    for (int k = 0; k < V; ++k) {
        if (!(r[k] > 0.f)) t[k] = 0;
        if (BOTH) w[k] = __uint_as_float((uint32_t)t[k] << 16);
    }
    *reinterpret_cast<vg*>(y + i) = t;
    if (BOTH) *reinterpret_cast<vf*>(y32 + i) = w;
}

// dst += src
__global__ void add_into_kernel(size_t n, const float* __restrict__ src, float* __restrict__ dst) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] += src[i];
}

// bfloat16 -> fp32 (exact: the bf16 bits are the upper half of the fp32 word)
__global__ void widen_bf16_kernel(size_t n, const uint16_t* __restrict__ src, float* __restrict__ dst) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = __uint_as_float((uint32_t)src[i] << 16);
}

// ==================================================================== host launchers


FoldArgs fold_args(int R, int kd, int nd, int H, const float* W, const float* w, float* wv, const float* w2, float* wv2) {
    const size_t lanes = (size_t)R * kd * (H > 1 ? H : 8);
    return FoldArgs{W, w, w2, R, kd, nd, H, wv, wv2, (int)blocks_for(lanes, 256)};
}

rgnn_status_t fold_weight(const FoldArgs& f, hipStream_t st) {
    if (f.nd % 32) RGNN_FAIL(RGNN_EUNSUPPORTED, "fold_weight: width %d is not a multiple of 32", f.nd);
    if (f.H > 1 && f.w2) RGNN_FAIL(RGNN_EUNSUPPORTED, "fold_weight: two vectors per relation are built for one head");
    KernelTimer kt(st, "fold_weight");
    hipLaunchKernelGGL(fold_weight_kernel, dim3(f.blocks), dim3(256), 0, st, f);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

rgnn_status_t segment_scalar_sum(int n, const int32_t* ptr, const LongList& lng, const int32_t* via, const float* val,
                                 int stride, int off, float* out, hipStream_t st, const char* label, int min_len,
                                 int heads, bool long_only, int ostride, const FoldArgs* with_fold) {
    FoldArgs fold = with_fold ? *with_fold : FoldArgs{};
    if (!fold_rides(fold)) {
        RGNN_TRY(fold_weight(fold, st));
        fold = FoldArgs{};
    }
    if (fold.blocks > 0 && (fold.nd % 32 || (fold.H > 1 && fold.w2))) RGNN_FAIL(RGNN_EUNSUPPORTED, "segment_scalar_sum: this fold is not built");
    if (heads < 1 || (heads & (heads - 1))) RGNN_FAIL(RGNN_EUNSUPPORTED, "segment_scalar_sum: the head count must be a power of two, got %d", heads);
    if (n == 0 || (long_only && lng.n == 0)) return fold.blocks > 0 ? fold_weight(fold, st) : RGNN_OK;
    KernelTimer kt(st, label);
    const size_t long_blocks = (size_t)lng.n * heads;
    if (ostride <= 0) ostride = heads;
    if (long_only) n = 0;   // only the first kind of workgroups: the caller has summed the segments of up to kSerialMax entries
    if ((heads == 2 || heads == 4) && stride % heads == 0 && off % heads == 0 && ostride % heads == 0) {
        const dim3 grid((unsigned)(lng.n + blocks_for((size_t)n, 256) + fold.blocks));
        if (heads == 2) hipLaunchKernelGGL(segment_vec_sum_kernel<2>, grid, dim3(256), 0, st, fold, n, ptr, via, val, stride, off, min_len, out, lng.n, lng.ids, ostride);
        else hipLaunchKernelGGL(segment_vec_sum_kernel<4>, grid, dim3(256), 0, st, fold, n, ptr, via, val, stride, off, min_len, out, lng.n, lng.ids, ostride);
        RGNN_CHECK_LAUNCH();
        return RGNN_OK;
    }
    hipLaunchKernelGGL(segment_scalar_sum_kernel, dim3((unsigned)(long_blocks + blocks_for((size_t)n * heads, 256) + fold.blocks)), dim3(256), 0, st, fold, n,
                       heads, ptr, via, val, stride, off, min_len, out, lng.n, lng.ids, ostride);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

rgnn_status_t edge_softmax(const rgnn_graph* g, const float* s_src, const float* s_dst, float slope, float* att,
                           float* part_m, float* part_s, hipStream_t st, float* ms) {
    const ItemList& L = g->dst_items;
    if (L.num_items == 0) return RGNN_OK;
    SoftmaxArgs a{dev_items(L), g->idx[RGNN_IDX_IN_PAIR], g->idx[RGNN_IDX_IN_RUN], s_src, s_dst, slope, att, part_m, part_s,
                  reinterpret_cast<float2*>(ms)};
    {
        KernelTimer kt(st, "edge_softmax");
        hipLaunchKernelGGL(edge_softmax_kernel, dim3(blocks_for((size_t)g->N, 256)), dim3(256), 0, st, a, (int)g->N,
                           g->idx[RGNN_IDX_IN_PTR]);
        RGNN_CHECK_LAUNCH();
        if (L.num_long > 0) {
            hipLaunchKernelGGL(edge_softmax_long_kernel, dim3(blocks_for((size_t)L.num_long * 64, 256)), dim3(256), 0, st,
                               a, L.num_long, L.long_item);
            RGNN_CHECK_LAUNCH();
        }
    }
    if (L.num_partials > 0) {
        KernelTimer kt(st, "edge_softmax.finish");
        hipLaunchKernelGGL(edge_softmax_finish_kernel, dim3(blocks_for((size_t)L.num_partials * 64, 256)), dim3(256), 0,
                           st, L.num_partials, L.part_item, L.part_split, L.split_ptr, dev_items(L), part_m, part_s, att,
                           reinterpret_cast<float2*>(ms));
        RGNN_CHECK_LAUNCH();
    }
    return RGNN_OK;
}

// Launches KERNEL<DD, ..., TI, TO> for the storage types of a call.  bf16 rows exist at width 128 only.
#define RGNN_DISPATCH_ROWS(D_, IN16, OUT16, ...)                                                         \
    do {                                                                                                 \
        if (!(IN16) && !(OUT16)) { using TI = float; using TO = float; RGNN_DISPATCH_D(D_, __VA_ARGS__); }      \
        else if ((D_) != 128) RGNN_FAIL(RGNN_EUNSUPPORTED, "bf16 rows need width 128, got %d", (int)(D_)); \
        else if ((IN16) && (OUT16)) { using TI = bf16_t; using TO = bf16_t; constexpr int DD = 128; __VA_ARGS__; } \
        else if (IN16) { using TI = bf16_t; using TO = float; constexpr int DD = 128; __VA_ARGS__; }            \
        else { using TI = float; using TO = bf16_t; constexpr int DD = 128; __VA_ARGS__; }                      \
    } while (0)

rgnn_status_t combine_softmax(const ItemList& L, int D, int H, const float* partial, const float* part_ms, void* out,
                              int out_bf16, float* ms, bool full_exp, int piece_len, const char* label, hipStream_t st, const int32_t* ms_row) {
    if (L.num_split == 0) return RGNN_OK;
    KernelTimer kt(st, label);
#define RGNN_COMBINE(HH, TO_, FULL_)                                                                                  \
    RGNN_DISPATCH_D(D, hipLaunchKernelGGL((combine_softmax_kernel<DD, (DD / (HH) >= 16 ? (HH) : 1), TO_, FULL_>), dim3(L.num_split), dim3(256), 0, st, \
                                          L.split_row, L.split_ptr, partial, reinterpret_cast<const float2*>(part_ms), \
                                          static_cast<TO_*>(out), reinterpret_cast<float2*>(ms), ms_row, piece_len))
#define RGNN_COMBINE_H(HH)                                                                                            \
    do {                                                                                                              \
        if (out_bf16) RGNN_COMBINE(HH, bf16_t, true);                                                                 \
        else if (full_exp) RGNN_COMBINE(HH, float, true);                                                             \
        else RGNN_COMBINE(HH, float, false);                                                                          \
    } while (0)
    if (H < 1 || D / H < 16) { if (H != 1) RGNN_FAIL(RGNN_EUNSUPPORTED, "combine_softmax: %d heads at width %d not built", H, D); }
    if (H == 1) RGNN_COMBINE_H(1);
    else if (H == 2) RGNN_COMBINE_H(2);
    else if (H == 4) RGNN_COMBINE_H(4);
    else if (H == 8) RGNN_COMBINE_H(8);
    else RGNN_FAIL(RGNN_EUNSUPPORTED, "combine_softmax: %d heads not built (1, 2, 4, 8)", H);
#undef RGNN_COMBINE_H
#undef RGNN_COMBINE
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

rgnn_status_t combine_partials(const ItemList& L, int D, const float* partial, void* out, int out_bf16, const char* label,
                               hipStream_t st, const Rank1* r1, int heads, int copies, size_t out_copy, const float* extra) {
    if (L.num_split == 0) return RGNN_OK;
    const Rank1 r1v = r1 ? *r1 : Rank1{nullptr, 0, nullptr, nullptr};
    KernelTimer kt(st, label);
#define RGNN_LAUNCH_COMBINE(DD_, TO_)                                                                                  \
    do {                                                                                                               \
        if (few_long_segments(L))                                                                                      \
            hipLaunchKernelGGL((combine_partials_kernel<DD_, TO_, 1024, 8>), dim3(L.num_split, copies, DD_ / 32), dim3(1024), 0, st, L.split_row, \
                               L.split_ptr, partial, static_cast<TO_*>(out), (size_t)L.num_partials * DD_, out_copy, r1v, (DD_ / 4) / heads, extra); \
        else                                                                                                           \
            hipLaunchKernelGGL((combine_partials_kernel<DD_, TO_, 256, DD_ / 4>), dim3(L.num_split, copies), dim3(256), 0, st, L.split_row, \
                               L.split_ptr, partial, static_cast<TO_*>(out), (size_t)L.num_partials * DD_, out_copy, r1v, (DD_ / 4) / heads, extra); \
    } while (0)
    if (D == 256) {
        if (out_bf16) RGNN_LAUNCH_COMBINE(256, bf16_t);
        else RGNN_LAUNCH_COMBINE(256, float);
    } else if (out_bf16) {
        RGNN_DISPATCH_D(D, RGNN_LAUNCH_COMBINE(DD, bf16_t));
    } else {
        RGNN_DISPATCH_D(D, RGNN_LAUNCH_COMBINE(DD, float));
    }
#undef RGNN_LAUNCH_COMBINE
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

rgnn_status_t gather_sum(const ItemList& L, int D, const int32_t* via, const int32_t* rowidx, int row_by_k,
                         const float* coef, int cstride, int cabs, const void* src, void* out, float* partial,
                         hipStream_t st, int role, const char* label, const char* combine_label, int heads,
                         int src_bf16, int out_bf16, const Rank1* r1, const float* extra) {
    if (L.num_items == 0) return RGNN_OK;
    const Rank1 r1v = r1 ? *r1 : Rank1{nullptr, 0, nullptr, nullptr};
    const int lpr = D / (src_bf16 ? 8 : 4);
    // enough short / single-entry segments to be worth launches of their own; the two ranges are adjacent
    const int ns = batched_count(L.num_single, current_schedule_flags());
    const int nsh = batched_count(L.num_short, current_schedule_flags());
    const int skip_first = nsh > 0 ? L.first_short : L.first_single;
    GatherArgs a{dev_items(L), via, rowidx, row_by_k, coef, cstride, cabs, lpr / heads, src, out, partial, skip_first, nsh + ns, r1v, nullptr, 1, heads, extra};
    if (extra && role != 3) RGNN_FAIL(RGNN_EUNSUPPORTED, "gather_sum: rows are added to the sums over sources only");
    {
        KernelTimer kt(st, label);
        GatherRanges r{};
        r.general_blocks = (int)blocks_for(L.num_items - nsh - ns, 256 / lpr);
        r.short_blocks = nsh > 0 ? (int)blocks_for((size_t)(nsh + 1) / 2, 256 / lpr) : 0;
        r.short_first = L.first_short; r.short_n = nsh; r.single_first = L.first_single; r.single_n = ns;
        const int single_blocks = ns > 0 ? (int)blocks_for((size_t)(ns + 3) / 4, 256 / lpr) : 0;
        const dim3 grid(r.general_blocks + r.short_blocks + single_blocks);
#define RGNN_LAUNCH_GATHER(KERNEL, GRID, ...)                                                                              \
    do {                                                                                                                   \
        if (role == 0) RGNN_DISPATCH_ROWS(D, src_bf16, out_bf16, hipLaunchKernelGGL((KERNEL<DD, 0, TI, TO>), GRID, dim3(256), 0, st, __VA_ARGS__)); \
        else if (role == 1) RGNN_DISPATCH_ROWS(D, src_bf16, out_bf16, hipLaunchKernelGGL((KERNEL<DD, 1, TI, TO>), GRID, dim3(256), 0, st, __VA_ARGS__)); \
        else RGNN_DISPATCH_ROWS(D, src_bf16, out_bf16, hipLaunchKernelGGL((KERNEL<DD, 2, TI, TO>), GRID, dim3(256), 0, st, __VA_ARGS__)); \
        RGNN_CHECK_LAUNCH();                                                                                               \
    } while (0)
        if (r1 && (src_bf16 || out_bf16 || role != 1)) RGNN_FAIL(RGNN_EUNSUPPORTED, "gather_sum: the rank-1 term is built for fp32 rows of the pair-major walk");
        if (r1) {
            if (grid.x > 0) {
                RGNN_DISPATCH_D(D, hipLaunchKernelGGL((gather_sum_kernel<DD, 1, float, float, true>), grid, dim3(256), 0, st, a, r));
                RGNN_CHECK_LAUNCH();
            }
        } else if (role == 3) {
            if (src_bf16 || out_bf16) RGNN_FAIL(RGNN_EUNSUPPORTED, "gather_sum: the sums over sources are built for fp32 rows");
            if (grid.x > 0) {
                RGNN_DISPATCH_D(D, hipLaunchKernelGGL((gather_sum_kernel<DD, 3, float, float>), grid, dim3(256), 0, st, a, r));
                RGNN_CHECK_LAUNCH();
            }
        } else if (!src_bf16) {
            if (grid.x > 0) RGNN_LAUNCH_GATHER(gather_sum_kernel, grid, a, r);
        } else {
            if (r.general_blocks > 0) RGNN_LAUNCH_GATHER(gather_general_kernel, dim3(r.general_blocks), a);
            if (nsh > 0) RGNN_LAUNCH_GATHER(gather_short_kernel, dim3(r.short_blocks), a, L.first_short, nsh);
            if (ns > 0) RGNN_LAUNCH_GATHER(gather_single_kernel, dim3(single_blocks), a, L.first_single, ns);
        }
#undef RGNN_LAUNCH_GATHER
    }
    return combine_partials(L, D, partial, out, out_bf16, combine_label, st, &r1v, heads, 1, 0, extra);
}

rgnn_status_t gather_heads_rows(const ItemList& L, int D, int H, int out_rows, const int32_t* via, const int32_t* rowidx,
                                int row_by_k, const float* coef, const float* src, float* out, float* partial,
                                hipStream_t st, const char* label, const char* combine_label) {
    if (L.num_items == 0) return RGNN_OK;
    GatherArgs a{dev_items(L), via, rowidx, row_by_k, coef, H, 0, 1, src, out, partial, 0, 0, Rank1{nullptr, 0, nullptr, nullptr}, nullptr, 1, 1};
    {
        KernelTimer kt(st, label);
        const dim3 grid(blocks_for(L.num_items, 256 / (D / 4)));
#define RGNN_LAUNCH_NH(NH_) RGNN_DISPATCH_D(D, hipLaunchKernelGGL((gather_heads_rows_kernel<DD, NH_>), grid, dim3(256), 0, st, a, out_rows, L.num_partials))
        if (H == 2) RGNN_LAUNCH_NH(2);
        else if (H == 4) RGNN_LAUNCH_NH(4);
        else if (H == 8) RGNN_LAUNCH_NH(8);
        else RGNN_FAIL(RGNN_EUNSUPPORTED, "gather_heads_rows: %d heads not built (2, 4, 8)", H);
#undef RGNN_LAUNCH_NH
        RGNN_CHECK_LAUNCH();
    }
    return combine_partials(L, D, partial, out, 0, combine_label, st, nullptr, 1, H, (size_t)out_rows * D);
}

rgnn_status_t rgat_bwd_walks(const rgnn_graph* g, const RgatBwdWalks& a, hipStream_t st) {
    const ItemList &L = g->pair_items_multi, &R = g->relrun_items;
    const int D = a.d_out, K = a.d_in, H = a.heads;
    if (L.num_single > 0) RGNN_FAIL(RGNN_EUNSUPPORTED, "rgat_bwd_walks: the list of the pairs with several edges has single-entry segments");
    const Rank1 r1 = a.ws ? Rank1{a.ds_src, a.ds_src_stride, g->idx[RGNN_IDX_PAIR_REL], a.ws} : Rank1{nullptr, 0, nullptr, nullptr};
    const int nsh = batched_count(L.num_short, current_schedule_flags());
    const GatherArgs pair{dev_items(L), g->idx[RGNN_IDX_OUT_EPOS], g->idx[RGNN_IDX_OUT_DST], 0, a.adz, 2 * H, 0, D / 4 / H, a.dOut, a.G,
                          a.pair_partial, L.first_short, nsh, r1, a.ds_src, a.ds_src_stride, H};
    const GatherArgs run{dev_items(R), g->idx[RGNN_IDX_RELRUN_IDX], g->relrun_dst, 0, a.ds_dst, H, 0, H > 1 ? 1 : K / 4, a.X, a.U,
                         a.run_partial, R.num_items, 0, Rank1{nullptr, 0, nullptr, nullptr}, nullptr, 1, 1};
    GatherRanges r{};
    r.general_blocks = (int)blocks_for((size_t)(L.num_items - nsh), 256 / (D / 4));
    r.short_blocks = nsh > 0 ? (int)blocks_for((size_t)(nsh + 1) / 2, 256 / (D / 4)) : 0;
    r.short_first = L.first_short; r.short_n = nsh;
    const int run_blocks = (int)blocks_for((size_t)R.num_items, 256 / (K / 4));
    const dim3 grid(run_blocks + r.general_blocks + r.short_blocks);
    if (grid.x > 0) {
        KernelTimer kt(st, "pair_run_walks");
#define RGNN_WALKS(D_, K_, H_) hipLaunchKernelGGL((pair_run_walks_kernel<D_, K_, H_>), grid, dim3(256), 0, st, pair, r, run, run_blocks, g->R, R.num_partials)
#define RGNN_WALKS_DK(H_)                                                                                    \
    do {                                                                                                     \
        if (D == 64 && K == 64) RGNN_WALKS(64, 64, H_);                                                      \
        else if (D == 32 && K == 32) RGNN_WALKS(32, 32, H_);                                                 \
        else if (D == 64 && K == 32) RGNN_WALKS(64, 32, H_);                                                 \
        else if (D == 32 && K == 64) RGNN_WALKS(32, 64, H_);                                                 \
        else RGNN_FAIL(RGNN_EUNSUPPORTED, "rgat_bwd_walks: widths %d -> %d not built", K, D);                \
    } while (0)
        if (H == 1 && D == 128 && K == 128) RGNN_WALKS(128, 128, 1);
        else if (H == 1) RGNN_WALKS_DK(1);
        else if (H == 2) RGNN_WALKS_DK(2);
        else if (H == 4) RGNN_WALKS_DK(4);
        else RGNN_FAIL(RGNN_EUNSUPPORTED, "rgat_bwd_walks: %d heads not built (1, 2, 4)", H);
#undef RGNN_WALKS_DK
#undef RGNN_WALKS
        RGNN_CHECK_LAUNCH();
    }
    return combine_partials(L, D, a.pair_partial, a.G, 0, "aggregate_bwd_pair.combine", st, &r1, H);
}

rgnn_status_t aggregate_edge_parallel(const rgnn_graph* g, int D, const float* att, const float* Hs, float* out,
                                      hipStream_t st) {
    if (g->N == 0) return RGNN_OK;
    KernelTimer kt(st, "aggregate_fwd_edge_parallel");
    const size_t n = (size_t)g->N * D;
    hipLaunchKernelGGL(zero_f32_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, out);   // a kernel, not a memset: callers may capture
    RGNN_CHECK_LAUNCH();
    if (g->E == 0) return RGNN_OK;
    RGNN_DISPATCH_D(D, hipLaunchKernelGGL(aggregate_edge_parallel_kernel<DD>, dim3(blocks_for(((size_t)g->E + kEdgeChunk - 1) / kEdgeChunk, 256 / (DD / 4))),
                                          dim3(256), 0, st, g->E, g->idx[RGNN_IDX_IN_PAIR], g->idx[RGNN_IDX_IN_RUN],
                                          g->idx[RGNN_IDX_RUN_DST], att, Hs, out));
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

rgnn_status_t node_grad_sum(const rgnn_graph* g, int D, const void* dXp, const float* ds_dst, const float* wtp,
                            const float* extra, void* dX, hipStream_t st, int in_bf16, int out_bf16, int heads,
                            const void* dXp2, const RgatFinish* finish) {
    RgatFinish fin = finish ? *finish : RgatFinish{};
    const int64_t fin_blocks = finish ? finish_blocks(fin.R, fin.kd, fin.nd) : 0;
    if (fin_blocks > INT32_MAX / 2) RGNN_FAIL(RGNN_EUNSUPPORTED, "node_grad_sum: the parameter gradients of %d relations are too many", fin.R);
    fin.blocks = (int)fin_blocks;
    if (finish && !ds_dst) RGNN_FAIL(RGNN_EINVAL, "node_grad_sum: the parameter gradients go with the run term");
    if (g->N == 0 && fin.blocks == 0) return RGNN_OK;
    if (ds_dst && dXp2) RGNN_FAIL(RGNN_EINVAL, "node_grad_sum: the run term and a second row tensor exclude each other");
    if (heads < 1 || (heads & (heads - 1))) RGNN_FAIL(RGNN_EUNSUPPORTED, "node_grad_sum: the head count must be a power of two, got %d", heads);
    NodeSumArgs a{dev_items(g->srcpair_items), g->idx[RGNN_IDX_SRCPAIR_IDX], dXp, dXp2,
                  g->idx[RGNN_IDX_DST_RUN_PTR], g->idx[RGNN_IDX_RUN_REL], ds_dst, wtp, extra, dX};
    if (ds_dst && (in_bf16 || out_bf16)) RGNN_FAIL(RGNN_EUNSUPPORTED, "node_grad_sum: the run term is built for fp32 rows");
    KernelTimer kt(st, "node_grad_sum");
    const dim3 grid = flat_grid((int64_t)blocks_for((size_t)g->N, 256 / (D / (in_bf16 ? 8 : 4))) + fin.blocks);
    if (ds_dst) {
#define RGNN_NODE_SUM(H_) RGNN_DISPATCH_D(D, hipLaunchKernelGGL((node_grad_sum_kernel<DD, float, float, H_, false>), grid, dim3(256), 0, st, a, fin))
        if (heads == 1) RGNN_NODE_SUM(1);
        else if (heads == 2) RGNN_NODE_SUM(2);
        else if (heads == 4) RGNN_NODE_SUM(4);
        else if (heads == 8) RGNN_NODE_SUM(8);
        else RGNN_FAIL(RGNN_EUNSUPPORTED, "node_grad_sum: %d heads not built (1, 2, 4, 8)", heads);
#undef RGNN_NODE_SUM
    } else if (dXp2 && (in_bf16 || out_bf16))
        RGNN_FAIL(RGNN_EUNSUPPORTED, "node_grad_sum: a second row tensor is built for fp32 rows");
    else if (dXp2)
        RGNN_DISPATCH_D(D, hipLaunchKernelGGL((node_grad_sum_kernel<DD, float, float, 0, true>), grid, dim3(256), 0, st, a, fin));
    else
        RGNN_DISPATCH_ROWS(D, in_bf16, out_bf16, hipLaunchKernelGGL((node_grad_sum_kernel<DD, TI, TO, 0, false>), grid, dim3(256), 0, st, a, fin));
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

template <int D, bool LDSW>
static rgnn_status_t launch_run_term(const rgnn_graph* g, const float* ds_dst, const float* wtp, float* dX, const RgatFinish& fin, hipStream_t st) {
    const size_t lds = std::max<size_t>(LDSW ? (size_t)g->R * D : 0, 512) * sizeof(float), groups = kRunTermThreads / (D / 4);
    const void* fn = reinterpret_cast<const void*>(run_term_kernel<D, LDSW>);
    RGNN_TRY(allow_dynamic_lds(fn, lds));
    int per_cu = 1;
    RGNN_TRY(resident_blocks_per_cu(fn, kRunTermThreads, lds, &per_cu));
    const ItemList& L = g->dstrun_items;
    const size_t blocks = std::min<size_t>(((size_t)L.num_items + groups - 1) / groups, (size_t)per_cu * g->num_cus);
    hipLaunchKernelGGL((run_term_kernel<D, LDSW>), dim3((unsigned)blocks + fin.blocks), dim3(kRunTermThreads), lds, st, dev_items(L), g->R,
                       g->idx[RGNN_IDX_DST_RUN_PTR], g->idx[RGNN_IDX_RUN_REL], ds_dst, wtp, dX, fin);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}
rgnn_status_t rgat_run_term(const rgnn_graph* g, int D, const float* ds_dst, const float* wtp, float* dX, RgatFinish fin, hipStream_t st) {
    const int64_t blocks = finish_blocks(fin.R, fin.kd, fin.nd);
    if (blocks > kMaxFinishBlocks) RGNN_FAIL(RGNN_EUNSUPPORTED, "run term: the parameter gradients of %d relations are too many", fin.R);
    fin.blocks = (int)blocks;
    KernelTimer kt(st, "run_term");
    if (sched_ws_in_lds(g->R, D)) RGNN_DISPATCH_D(D, return (launch_run_term<DD, true>(g, ds_dst, wtp, dX, fin, st)));
    else RGNN_DISPATCH_D(D, return (launch_run_term<DD, false>(g, ds_dst, wtp, dX, fin, st)));
}

rgnn_status_t widen_bf16(size_t n, const uint16_t* src, float* dst, hipStream_t st) {
    if (n == 0) return RGNN_OK;
    KernelTimer kt(st, "widen_bf16");
    hipLaunchKernelGGL(widen_bf16_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, src, dst);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}
rgnn_status_t add_into(size_t n, const float* src, float* dst, hipStream_t st) {
    if (n == 0) return RGNN_OK;
    KernelTimer kt(st, "add_into");
    hipLaunchKernelGGL(add_into_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, src, dst);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}
rgnn_status_t relu_inplace(size_t n, float* x, hipStream_t st) {
    if (n == 0) return RGNN_OK;
    KernelTimer kt(st, "relu");
    hipLaunchKernelGGL(relu_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, x);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}
rgnn_status_t relu_grad(size_t n, const float* ref, const void* gin, void* y, hipStream_t st, int bf16, float* y32) {
    if (n == 0) return RGNN_OK;
    if (y32 && !bf16) RGNN_FAIL(RGNN_EUNSUPPORTED, "relu_grad: the fp32 copy is for bf16 gradients");
    KernelTimer kt(st, "relu_grad");
    // four elements per thread where every tensor allows it (ref and gin are the caller's)
    const bool four = n % 4 == 0 && ((reinterpret_cast<uintptr_t>(ref) | reinterpret_cast<uintptr_t>(gin) | reinterpret_cast<uintptr_t>(y) |
                                      reinterpret_cast<uintptr_t>(y32)) & 15) == 0;
#define RGNN_RELU_GRAD(G_, BOTH_)                                                                                       \
    do {                                                                                                               \
        if (four)                                                                                                      \
            hipLaunchKernelGGL((relu_grad_kernel<G_, BOTH_, 4>), dim3(blocks_for(n / 4, 256)), dim3(256), 0, st, n, ref, \
                               static_cast<const G_*>(gin), static_cast<G_*>(y), y32);                                 \
        else                                                                                                           \
            hipLaunchKernelGGL((relu_grad_kernel<G_, BOTH_, 1>), dim3(blocks_for(n, 256)), dim3(256), 0, st, n, ref,   \
                               static_cast<const G_*>(gin), static_cast<G_*>(y), y32);                                 \
    } while (0)
    if (!bf16) RGNN_RELU_GRAD(float, false);
    else if (y32) RGNN_RELU_GRAD(uint16_t, true);
    else RGNN_RELU_GRAD(uint16_t, false);
#undef RGNN_RELU_GRAD
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

}  // namespace rgnn
