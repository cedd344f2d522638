// Layer entry points of the C ABI: argument checks, carving of the caller's workspace, and
// the sequence of kernel launches that makes up each layer.  No allocation, no
// synchronisation; everything is enqueued on the caller's stream.
#include "rgnn_internal.h"
#include "traversal.h"
#include "schedule.h"

#include <map>
#include <mutex>

using namespace rgnn;

namespace {

// Bump allocator over a caller-provided buffer; with base == nullptr it only measures.
struct Carver {
    char* base;
    size_t off = 0;
    explicit Carver(void* b) : base(static_cast<char*>(b)) {}
    template <typename Tv>
    Tv* take(size_t n) {
        Tv* p = base ? reinterpret_cast<Tv*>(base + off) : nullptr;
        off += align_up(std::max<size_t>(n, 1) * sizeof(Tv));
        return p;
    }
    // n elements of a row tensor stored as bf16 (half) or fp32
    void* rows(size_t n, bool half) { return half ? static_cast<void*>(take<uint16_t>(n)) : static_cast<void*>(take<float>(n)); }
};

// bfloat16 workloads at width 128 keep every row tensor (inputs, intermediates, saved tensors,
// incoming gradients) in bf16 storage and run the typed linears on the bf16 matrix cores; sums
// and products are fp32, results handed back to the caller are fp32.  At the other widths the
// bf16 inputs are widened once and the fp32 kernels run on the copies.
inline bool rows_bf16(const rgnn_layer_desc_t* d) { return d->dtype == RGNN_BF16 && d->d_out == 128; }

// bfloat16 inputs that an fp32 kernel consumes are widened to fp32 in a staging area that
// follows the regular carve-out of the workspace.
struct Bf16Stage {
    Carver c;
    bool on;
    hipStream_t st;
    rgnn_status_t status = RGNN_OK;
    Bf16Stage(void* ws, size_t carved, bool bf16, hipStream_t s)
        : c(ws ? static_cast<char*>(ws) + carved : nullptr), on(bf16), st(s) {}
    // returns the fp32 view of `p` (n elements): p itself for fp32 input, the widened copy for bf16
    const float* in(const void* p, size_t n) {
        if (!on || !p) return static_cast<const float*>(p);
        float* d = c.take<float>(n);
        if (c.base && status == RGNN_OK) status = widen_bf16(n, static_cast<const uint16_t*>(p), d, st);
        return d;
    }
    void reserve(size_t n) { if (on) (void)c.take<float>(n); }
};

// A [num_nodes, d] tensor may be NULL when the graph has no nodes.
inline bool missing(const rgnn_graph_t* g, const void* p) { return !p && g->N > 0; }
inline bool overlap(const void* p, size_t np, const void* q, size_t nq) {
    return reinterpret_cast<uintptr_t>(p) < reinterpret_cast<uintptr_t>(q) + nq && reinterpret_cast<uintptr_t>(q) < reinterpret_cast<uintptr_t>(p) + np;
}

rgnn_status_t check_desc(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, int layer) {
    if (!g || !d) RGNN_FAIL(RGNN_EINVAL, "graph or desc is NULL");
    if (d->flags & ~RGNN_FLAG_ALL) RGNN_FAIL(RGNN_EINVAL, "unknown bits in desc.flags");
    if ((d->flags & (RGNN_FLAG_EDGE_PARALLEL_AGGREGATION | RGNN_FLAG_SEPARATE_SOFTMAX)) && (layer != RGNN_LAYER_RGAT || d->heads != 1))
        RGNN_FAIL(RGNN_EUNSUPPORTED, "the edge-parallel aggregation and the separate softmax pass are schedules of single-head RGAT only");
    if (d->dtype != RGNN_F32 && d->dtype != RGNN_BF16) RGNN_FAIL(RGNN_EINVAL, "unknown dtype %d", d->dtype);
    // widths: 32, 64 or 128 on both sides; RGCN and RGAT with fp32 inputs also take 32 -> 64 and 64 -> 32
    const bool w_in = d->d_in == 32 || d->d_in == 64 || d->d_in == 128, w_out = d->d_out == 32 || d->d_out == 64 || d->d_out == 128;
    const bool mixed_ok = layer != RGNN_LAYER_HGT && d->dtype == RGNN_F32 && d->d_in <= 64 && d->d_out <= 64;
    if (!w_in || !w_out || (d->d_in != d->d_out && !mixed_ok))
        RGNN_FAIL(RGNN_EUNSUPPORTED, "need d_in == d_out in {32, 64, 128} (RGCN / RGAT with fp32 inputs: also 32 -> 64 and 64 -> 32), got %d -> %d",
                  d->d_in, d->d_out);
    if (layer == RGNN_LAYER_RGAT) {
        if (d->heads < 1 || d->d_out % d->heads != 0) RGNN_FAIL(RGNN_EINVAL, "heads must divide d_out");
        const int dh = d->d_out / d->heads;
        if (d->heads > 1 && dh != 16 && dh != 32 && dh != 64)
            RGNN_FAIL(RGNN_EUNSUPPORTED, "multi-head RGAT needs d_out / heads in {16, 32, 64}, got %d", dh);
        if (std::max<int64_t>(g->N, g->E) * d->heads > INT32_MAX)
            RGNN_FAIL(RGNN_EUNSUPPORTED, "multi-head RGAT needs num_nodes * heads and num_edges * heads < 2^31");
    }
    // with the widths and head widths allowed above the head count is a power of two; the kernels index with shifts
    if ((layer == RGNN_LAYER_RGAT || layer == RGNN_LAYER_HGT) && (d->heads & (d->heads - 1)))
        RGNN_FAIL(RGNN_EUNSUPPORTED, "the head count must be a power of two, got %d", d->heads);
    if (layer == RGNN_LAYER_RGAT && !(d->slope >= 0.f && d->slope <= 1.f))
        RGNN_FAIL(RGNN_EINVAL, "leaky-ReLU slope must be in [0, 1]");
    if (layer == RGNN_LAYER_RGCN) {
        if (d->norm != RGNN_NORM_NONE && d->norm != RGNN_NORM_IN_DEGREE_PER_REL) RGNN_FAIL(RGNN_EINVAL, "unknown norm %d", d->norm);
        if (d->activation != RGNN_ACT_NONE && d->activation != RGNN_ACT_RELU) RGNN_FAIL(RGNN_EINVAL, "unknown activation %d", d->activation);
    }
    if (layer == RGNN_LAYER_HGT) {
        if (d->heads < 1 || d->d_out % d->heads != 0) RGNN_FAIL(RGNN_EINVAL, "heads must divide d_out");
        const int dh = d->d_out / d->heads;
        if (dh != 16 && dh != 32 && dh != 64) RGNN_FAIL(RGNN_EUNSUPPORTED, "HGT needs d_out / heads in {16, 32, 64}, got %d", dh);
        if (std::max<int64_t>(g->N, g->E) * d->heads > INT32_MAX)
            RGNN_FAIL(RGNN_EUNSUPPORTED, "HGT needs num_nodes * heads and num_edges * heads < 2^31");
    }
    return RGNN_OK;
}

// ---- RGNN_FLAG_ACCUMULATE ---------------------------------------------------------------
// The input gradient is accumulated by the kernel that writes it (it reads the row it is about to store).  The
// parameter gradients are small and written by many different kernels, so under the flag they are formed in
// workspace buffers of their own and added to the caller's at the end of the call.
inline bool grads_accumulate(const rgnn_layer_desc_t* d) { return (d->flags & RGNN_FLAG_ACCUMULATE) != 0; }
struct GradAcc {
    static constexpr int kMax = 8;
    int n = 0;
    float* tmp[kMax];
    float* dst[kMax];
    size_t len[kMax];
    // where the backward pass is to write this gradient: the workspace buffer if there is one, else the caller's
    void* route(float* tmp_buf, void* dst_buf, size_t count) {
        if (!tmp_buf || !dst_buf) return dst_buf;
        tmp[n] = tmp_buf; dst[n] = static_cast<float*>(dst_buf); len[n] = count; ++n;
        return tmp_buf;
    }
    rgnn_status_t flush(hipStream_t st) const {
        for (int i = 0; i < n; ++i) RGNN_TRY(add_into(len[i], tmp[i], dst[i], st));
        return RGNN_OK;
    }
};

// The chunkings of one list of row tiles that the typed linears pick from:
//   many, wide  bf16 inputs, forward with fp32 results or an fp32 operand: weight in bf16 / an fp32 weight to be split
//   f32         the fp32 forward: one resident round, of three workgroups per compute unit up to width 64, of one at width 128
//   cu2         bf16 rows on both sides, forward and backward with one bf16 weight: two workgroups per compute unit
//   cu1         the bf16 forward and backward with two weights, the backward with a split one, and the fp32 one at width 128: one workgroup per compute unit
//   f32_bwd     the fp32 backward.  Up to width 64 it fills a compute unit's LDS, and one chunk per compute unit saves the weight
//               loads, flushes and slots of three rounds of shorter ones (62 us for 48 at 141k pairs and 108 for 82 at 349k, the
//               same within 1 % at 7.3M).  But where relations are short a chunk is a row of runs (segments), each with a load, one
//               or two rounds of units and a flush, and its length depends on how many: then the dispatcher has to even out the
//               chunks of `wide`.  Pairs of relations with Zipf 1.2 frequencies, cu1 / wide, width 64: 0.91, 0.93 and 0.98 of the
//               time with 1.7 runs per chunk (200k, 1M and 4M edges), 1.18, 1.02 and 1.03 with 2.1, 1.13 to 1.11 with 2.8 to 2.9;
//               with Zipf 1.0 the lines cross at 2.5.  With five tiles per chunk or fewer cu1 wins at any number of runs
//               (0.78 to 0.97 at 40k and 70k edges; 1.00 to 1.11 with six to eight tiles and two to four runs).
struct Chunkings {
    const rgnn::TileList* many; const rgnn::TileList* wide; const rgnn::TileList* f32; const rgnn::TileList* f32_bwd; const rgnn::TileList* cu2;
    const rgnn::TileList* cu1;
};
inline Chunkings chunkings(const rgnn::TileList& many, const rgnn::TileList& wide, const rgnn::TileList& cu2, const rgnn::TileList& cu1, int width) {
    const bool few_runs = 8 * (int64_t)cu1.num_slots <= 15 * (int64_t)cu1.num_chunks || cu1.num_tiles <= 5 * cu1.num_chunks;
    return {&many, &wide, width == 128 ? &cu1 : &wide, width == 128 || few_runs ? &cu1 : &wide, &cu2, &cu1};
}
inline Chunkings pair_chunks(const rgnn_graph_t* g, int width) {
    return chunkings(g->pair_tiles, g->pair_tiles_wide, g->pair_tiles_cu2, g->pair_tiles_cu1, width);
}
inline Chunkings node_chunks(const rgnn_graph_t* g, int width) {
    return chunkings(g->node_tiles, g->node_tiles_wide, g->node_tiles_cu2, g->node_tiles_cu1, width);
}
// rows per run instead of per pair (fp32 only: neither many nor cu2)
inline Chunkings run_chunks(const rgnn_graph_t* g, int width) {
    return chunkings(g->run_tiles_wide, g->run_tiles_wide, g->run_tiles_cu1, g->run_tiles_cu1, width);
}
inline const rgnn::TileList* all_chunks(const rgnn_graph_t* g, int width) { return width == 128 ? &g->all_tiles_cu1 : &g->all_tiles; }
// floats of scratch a backward typed linear needs on a list
size_t tl_bwd_scratch(bool rows16, const Chunkings& t, int d_in, int d_out) {
    if (!rows16) return typed_linear_bwd_scratch_floats(d_in, d_out, *t.f32_bwd);
    return (size_t)d_in * d_out * std::max((size_t)t.cu2->num_slots, 2 * (size_t)t.cu1->num_slots);
}

// ---- RGAT buffers -----------------------------------------------------------------------
// Hs, the destination halves of the logits per (run, head) and (max, sum) of every (destination, head) softmax.
struct RgatSaved { float* Hs; float* s_dst; float* ms; };
struct RgatFwdWs { float* wtp; float* s_src; float* att; float* part_m; float* part_s; float* part_ms; float* partial; };
struct RgatBwdWs {
    float* wtp; float* wsp; float* adz; float* ds_dst; float* ds_src; float* G; float* dXp; float* A; float* U;
    float* tl_part; float* partial; float* run_partial;
    float* acc_dW; float* acc_dws; float* acc_dwt;      // RGNN_FLAG_ACCUMULATE: the parameter gradients of this call
    float* Hs;                                          // where `saved` is laid out for rows per run: the message rows, formed again
};
// Rows per run (one head): Y[Q] product rows, A and lq as rgat_run_inputs leaves them (with the pieces of its cut runs), wsp = W w_s.
// All of it lies in `saved`, so that the forward's scratch is no larger than that of the rows per pair.
// What a graph and a descriptor without its flags say decides how a kept `saved` is laid out, so that a backward may carry other flags
// than its forward: a forward that a flag gives rows per pair leaves there what the rows per run need as well, and such a
// backward forms its message rows again.
struct RgatRunSaved { float* Y; float* s_dst; float* ms; float* A; float* lq; float* wsp; float* wtp; float* partial; float* part_ms; };
struct RgatRunBwdWs {
    float* dH; float* weight; float* rowdot; float* stat; float* dz; float* ds_dst; float* ds_src; float* A; float* U; float* tl_part; float* partial; float* a_partial;
    float* u_partial; float* acc_dW; float* acc_dws; float* acc_dwt;
};
inline bool rgat_keeps_runs(const rgnn_graph_t* g, const rgnn_layer_desc_t* d) {
    return sched_rgat_run_rows(g->run_rows, d->heads, g->R, g->E, d->d_out, 0) && sched_run_widths(d->d_in, d->d_out, g->E, g->rows_saved);
}
inline bool rgat_run_rows(const rgnn_graph_t* g, const rgnn_layer_desc_t* d) {
    return sched_use_run_rows(rgat_keeps_runs(g, d), d->flags);
}
// kept: s_dst and ms lie where the rows per pair have them, with Y and A in the place of Hs as far as they fit
size_t carve_rgat_run_saved(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, void* base, RgatRunSaved* s, bool kept) {
    Carver c(base);
    const size_t Q = g->Q, M = g->num_multi_runs, rk = (size_t)g->R * d->d_in, parts = g->multi_run_items.num_partials;
    const size_t room = kept ? (size_t)g->P * d->d_out : 0;
    if (kept) c.take<float>(room);
    s->s_dst = c.take<float>(Q);
    s->ms = c.take<float>(2 * (size_t)g->N);
    size_t used = 0;
    auto rows = [&](size_t n) {
        if (n > room - used) return c.take<float>(n);
        float* const p = base ? static_cast<float*>(base) + used : nullptr;
        used += n;
        return p;
    };
    s->Y = rows(Q * d->d_out);
    s->A = rows(M * d->d_in);
    s->lq = c.take<float>(2 * Q);
    s->wsp = c.take<float>(rk);
    s->wtp = c.take<float>(rk);
    s->partial = c.take<float>(parts * d->d_in);
    s->part_ms = c.take<float>(2 * parts);
    return c.off;
}
size_t carve_rgat_run_bwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, void* base, RgatRunBwdWs* w) {
    Carver c(base);
    const size_t Q = g->Q, rk = (size_t)g->R * d->d_in, rd = (size_t)g->R * d->d_out;
    w->dH = c.take<float>(Q * d->d_in);
    w->weight = c.take<float>(Q);
    w->rowdot = c.take<float>(Q);
    w->stat = c.take<float>(4 * Q);
    w->dz = c.take<float>((size_t)g->E);
    w->ds_dst = c.take<float>(Q);
    w->ds_src = c.take<float>((size_t)g->P);
    w->A = c.take<float>(rk);
    w->U = c.take<float>(rk);
    w->tl_part = c.take<float>(typed_linear_bwd_scratch_floats(d->d_in, d->d_out, *run_chunks(g, d->d_out).f32_bwd));
    w->partial = c.take<float>((size_t)g->src_items.num_partials * d->d_in);
    w->a_partial = c.take<float>((size_t)g->pair_blocks.num_partials * d->d_in);
    w->u_partial = c.take<float>((size_t)g->run_blocks.num_partials * d->d_in);
    const bool acc = grads_accumulate(d);
    w->acc_dW = acc ? c.take<float>(rk * d->d_out) : nullptr;
    w->acc_dws = acc ? c.take<float>(rd) : nullptr;
    w->acc_dwt = acc ? c.take<float>(rd) : nullptr;
    return c.off;
}
// RGAT with one head, and up to width 64 with two or four: the gradient rows of single-edge pairs are not written per
// pair; the typed-linear backward reads att_e * dOut[dst_e] through its row selector.
inline bool rgat_row_select(const rgnn_layer_desc_t* d) { return sched_row_select(RGNN_LAYER_RGAT, d->dtype, d->d_out, d->heads, 0, 0, 0, d->flags); }
inline bool rgat_edge_parallel(const rgnn_layer_desc_t* d) { return (d->flags & RGNN_FLAG_EDGE_PARALLEL_AGGREGATION) != 0; }
inline bool rgat_fused(const rgnn_layer_desc_t* d) { return sched_fused_softmax(d->flags); }

size_t carve_rgat_saved(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, void* base, RgatSaved* s) {
    Carver c(base);
    s->Hs = c.take<float>((size_t)g->P * d->d_out);
    s->s_dst = c.take<float>((size_t)g->Q * d->heads);
    s->ms = c.take<float>(2 * (size_t)g->N * d->heads);
    return c.off;
}
size_t carve_rgat_fwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, void* base, RgatFwdWs* w) {
    Carver c(base);
    const size_t H = d->heads, parts = (size_t)g->dst_items.num_partials;
    w->wtp = c.take<float>(H * g->R * d->d_in);
    w->s_src = w->att = w->part_m = w->part_s = w->part_ms = nullptr;
    if (!rgat_fused(d)) {
        // the comparison schedules (one head): per-pair source logits, a softmax pass of its own, attention weights per edge
        w->s_src = c.take<float>((size_t)g->P);
        w->att = c.take<float>((size_t)g->E);
        w->part_m = c.take<float>(parts);
        w->part_s = c.take<float>(parts);
        w->part_ms = w->part_m;              // (rows per run: both together)
    } else {
        w->part_ms = c.take<float>(2 * parts * H);
    }
    w->partial = c.take<float>(parts * d->d_out);
    return c.off;
}
size_t carve_rgat_bwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, void* base, RgatBwdWs* w) {
    Carver c(base);
    const size_t H = d->heads;
    w->wtp = c.take<float>(H * g->R * d->d_in);
    w->wsp = c.take<float>((size_t)g->R * d->d_in);
    w->adz = c.take<float>((size_t)g->E * 2 * H);                    // per edge: att per head, then dz per head
    w->ds_dst = c.take<float>((size_t)g->Q * H);
    // with the row selector: (ds_src[p], att of the pair's only edge) interleaved, one pair of floats per p
    //   (several heads: 2 H floats per p, ds_src[p][0..H) then, for a pair with one edge, that edge's att[0..H))
    w->ds_src = c.take<float>(2 * (size_t)g->P * H);
    w->G = c.take<float>((size_t)g->P * d->d_out);
    w->dXp = c.take<float>((size_t)g->P * d->d_in);
    w->A = c.take<float>(H * g->R * d->d_in);
    w->U = c.take<float>(H * g->R * d->d_in);
    w->tl_part = c.take<float>(typed_linear_bwd_scratch_floats(d->d_in, d->d_out, *pair_chunks(g, d->d_out).f32_bwd, (int)H));
    const size_t parts = std::max<size_t>({(size_t)g->pair_items.num_partials, (size_t)g->pair_items_multi.num_partials,
                                           (size_t)g->relpair_items.num_partials});
    w->partial = c.take<float>(parts * d->d_out);
    w->run_partial = c.take<float>((size_t)g->relrun_items.num_partials * d->d_in * H);   // one partial row per head
    const bool acc = grads_accumulate(d);
    w->acc_dW = acc ? c.take<float>((size_t)g->R * d->d_in * d->d_out) : nullptr;
    w->acc_dws = acc ? c.take<float>((size_t)g->R * d->d_out) : nullptr;
    w->acc_dwt = acc ? c.take<float>((size_t)g->R * d->d_out) : nullptr;
    w->Hs = rgat_keeps_runs(g, d) ? c.take<float>((size_t)g->P * d->d_out) : nullptr;
    return c.off;
}

// ---- RGCN buffers -----------------------------------------------------------------------
// Rows per run: A[m] = the mean (sum) of the input rows of the m-th run with several edges; Hs holds a message row per run.
struct RgcnFwdWs { void* Hs; float* partial; float* A; };
// A forward that is one launch goes with rows per pair in the backward: for rows per run it would have to form the sums as well.  Forward +
// backward, us, pairs / runs: 3000 nodes, 4 relations, 260k edges, 32 x 32 35 / 44, 64 x 64 47 / 65; 2000, 8, 140k, 64 x 64 41 / 53; 2000, 16, 300k,
// 32 x 64 47 / 52 (but 80 destinations, 8 relations, 140k edges, 64 x 64 67 / 56).  loop: with a self-loop.
inline bool rgcn_small(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, bool loop, uint32_t flags) {
    return sched_rgcn_small(d->dtype, d->d_in, d->d_out, loop, g->Q, g->N, g->dst_items.num_split > 0, g->longest_chain.runs, g->longest_chain.edges, flags);
}
// Whether `saved` holds the sums; whatever the flags: the backward may carry others than its forward.
inline bool rgcn_keeps_sums(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, bool loop) {
    return !rows_bf16(d) && sched_rgcn_run_rows(g->run_rows, g->E, d->d_out, 0) && sched_run_widths(d->d_in, d->d_out, g->E, g->rows_saved) &&
           !rgcn_small(g, d, loop, 0);
}
inline bool rgcn_run_rows(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, bool loop) { return sched_use_run_rows(rgcn_keeps_sums(g, d, loop), d->flags); }
size_t carve_rgcn_saved(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, bool loop, void* base, float** A) {
    Carver c(base);
    if (rgcn_keeps_sums(g, d, loop)) *A = c.take<float>((size_t)g->num_multi_runs * d->d_in);
    return c.off;
}
struct RgcnBwdWs { float* A; void* dPre; float* dPre32; void* G; void* dXp; float* dX0; float* tl_part; float* loop_part; float* partial; float* acc_dW; float* acc_dW0; };

size_t carve_rgcn_fwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, bool loop, void* base, RgcnFwdWs* w) {
    Carver c(base);
    // (a call without `saved` may take either plan and has to keep A here)
    const bool runs = rgcn_run_rows(g, d, loop);
    w->Hs = c.rows((size_t)(runs ? std::max(g->P, g->Q) : g->P) * d->d_out, rows_bf16(d));
    w->partial = c.take<float>(std::max({(size_t)g->dst_items.num_partials * d->d_out, runs ? (size_t)g->dstrun_items.num_partials * d->d_out : 0,
                                         rgcn_keeps_sums(g, d, loop) ? (size_t)g->multi_run_items.num_partials * d->d_in : 0}));
    w->A = runs ? c.take<float>((size_t)g->num_multi_runs * d->d_in) : nullptr;
    return c.off;
}
// RGCN with a self-loop, fp32 up to width 64: its backward runs with the pairs', where the pairs' chunks are one per compute unit
// (see Chunkings; with many short relations they stay apart).
inline bool rgcn_loop_bwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* d) {
    if (rgcn_run_rows(g, d, true)) return d->d_in <= 64 && d->d_out <= 64 && run_chunks(g, d->d_out).f32_bwd == &g->run_tiles_cu1;
    return d->d_in <= 64 && d->d_out <= 64 && pair_chunks(g, d->d_out).f32_bwd == &g->pair_tiles_cu1;
}
size_t carve_rgcn_bwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, bool loop, void* base, RgcnBwdWs* w) {
    Carver c(base);
    const bool h = rows_bf16(d), relu = d->activation == RGNN_ACT_RELU;
    w->dPre = c.rows(relu ? (size_t)g->N * d->d_out : 0, h);
    w->dPre32 = c.take<float>(relu && h ? (size_t)g->N * d->d_out : 0);   // fp32 copy for the self-loop kernels
    const bool runs = rgcn_run_rows(g, d, loop);
    w->G = runs ? nullptr : c.rows((size_t)g->P * d->d_out, h);
    w->dXp = c.rows((size_t)(runs ? g->Q : g->P) * d->d_in, h);        // (a row per run or per pair)
    w->A = runs ? c.take<float>((size_t)g->num_multi_runs * d->d_in) : nullptr;
    w->dX0 = c.take<float>((size_t)g->N * d->d_in);
    const bool with_loop = loop && rgcn_loop_bwd(g, d);
    w->tl_part = c.take<float>(std::max(tl_bwd_scratch(h, runs ? run_chunks(g, d->d_out) : pair_chunks(g, d->d_out), d->d_in, d->d_out),
                                        with_loop ? typed_linear_bwd_scratch_floats(d->d_in, d->d_out, runs ? g->run_tiles_loop : g->pair_tiles_loop) : 0));
    w->loop_part = c.take<float>(std::max(typed_linear_bwd_scratch_floats(d->d_in, d->d_out, g->all_tiles_cu1),
                                          with_loop ? typed_linear_bwd_scratch_floats(d->d_in, d->d_out, runs ? g->all_tiles_run_loop : g->all_tiles_loop) : 0));
    w->partial = c.take<float>(runs ? (size_t)std::max(g->src_items.num_partials, g->multi_run_items.num_partials) * d->d_in
                                    : (size_t)g->pair_items.num_partials * d->d_out);
    const bool acc = grads_accumulate(d);
    w->acc_dW = acc ? c.take<float>((size_t)g->R * d->d_in * d->d_out) : nullptr;
    w->acc_dW0 = acc ? c.take<float>((size_t)d->d_in * d->d_out) : nullptr;
    return c.off;
}

// ---- HGT buffers ------------------------------------------------------------------------
// Row tensors (void*) are bf16 when rows_bf16(desc), fp32 otherwise.
// Folded path (the graph ties every relation to one source node type): the key and message linears
// of the nodes are folded into the per-relation weights (Wf = Wk[type] Watt[r], Wv[type] Wmsg[r]), so
// K, V and their gradients do not exist and the per-pair rows come straight from X.
inline bool hgt_folded(const rgnn_graph_t* g, const rgnn_layer_desc_t* d) { return sched_hgt_folded(g->rel_src_tied, d->flags); }
// The sum over a node's pairs goes with the query's product of the node (rows in bf16).
inline bool hgt_pairs_with_query(const rgnn_graph_t* g, const rgnn_layer_desc_t* d) {
    return hgt_folded(g, d) && rows_bf16(d) && sched_hgt_pairs_with_query(g->N, g->P, g->max_node_pairs);
}
// folded path, fp32 rows up to width 64: the backwards of the two pair linears and of the query linear in one launch.  Backward of the
// layer with one launch / a launch each, width 64: 30 relations 100 / 123 us at 100k edges, 706 / 752 at 1.5M; 500 of equal frequency
// 292 / 297 at 20k, 583 / 644 at 400k; 1500 871 / 892 at 100k, 2005 / 2022 at 1.5M.
inline bool hgt_bwd_jobs(const rgnn_graph_t* g, const rgnn_layer_desc_t* d) { return hgt_folded(g, d) && d->d_out <= 64; }
// Its lists: one chunk per compute unit for all three; where relations are short (see Chunkings) and the chunks uneven, the lists of
// launches of their own.  Backward of the layer, us, shares / own lists, width 64, Zipf 1.1: 800 relations 843 / 717 at 400k edges, 2000 1098
// / 1087 at 100k, 2122 / 1676 at 1M, 4170 / 3586 at 4M; equal frequencies, whose chunks are even: 400 297 / 327 at 100k, 2000 1768 / 1821 at 1M.
inline bool hgt_own_lists(const rgnn_graph_t* g, int D) {
    const Chunkings c = pair_chunks(g, D);
    return c.f32_bwd != c.cu1 && g->pair_tiles_hgt.uneven();
}
inline const TileList* hgt_pair_list(const rgnn_graph_t* g, int D) { return hgt_own_lists(g, D) ? pair_chunks(g, D).f32_bwd : &g->pair_tiles_hgt; }
inline const TileList* hgt_node_list(const rgnn_graph_t* g, int D) { return hgt_own_lists(g, D) ? node_chunks(g, D).f32_bwd : &g->node_tiles_hgt; }
// The forward's products of one launch: one chunk per compute unit and list, or three where relations are short and the chunks uneven or
// many runs long.  Forward of the layer, us, one / three, width 64 (32), Zipf 1.1: 400 relations 97 / 91 (54 / 48) at 100k edges, 2000 620 / 472 (272
// / 202) at 1M, 1710 / 1438 at 4M; equal frequencies: 400 78 / 84 (50 / 48) at 100k, 1500 149 / 147 (72 / 64), 2000 443 / 439 at 1M.
inline const TileList* jobs_fwd_list(const Chunkings& c) {
    return c.f32_bwd != c.cu1 && (c.cu1->uneven() || c.cu1->num_slots >= 6 * (int64_t)c.cu1->num_chunks) ? c.wide : c.cu1;
}
// KM holds the key row and the message row of a pair side by side; ms the (max, sum) of every (destination, head) softmax.
struct HgtSaved { void* K; void* Q; void* V; void* Z; void* KM; float* ms; void* Wf_att; void* Wf_msg; };
struct HgtFwdWs { float* Wbd_att; float* Wbd_msg; float* part_ms; float* partial; };
struct HgtBwdWs {
    float* Wbd_att; float* Wbd_msg; float* dWbd_att; float* dWbd_msg; float* dWf_att;
    float* dWf_msg; void* dZ; float* adl; void* dKM;
    void* dQ; void* dKp; void* dVp; void* dK; void* dV; float* dXk; float* dXq; float* dXv; float* node_part[3]; float* pair_part[2];
    float* partial;
    float* acc_node[4]; float* acc_rel[2]; float* acc_mu;     // RGNN_FLAG_ACCUMULATE: dWk, dWq, dWv, dWo; dWatt, dWmsg; dmu
};

size_t carve_hgt_saved(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, void* base, HgtSaved* s) {
    Carver c(base);
    const bool h = rows_bf16(d);
    const size_t nd = (size_t)g->N * d->d_out, pd = (size_t)g->P * d->d_out, kv = hgt_folded(g, d) ? 0 : nd;
    s->K = c.rows(kv, h); s->Q = c.rows(nd, h); s->V = c.rows(kv, h); s->Z = c.rows(nd, h);
    s->KM = c.rows(2 * pd, h);
    s->ms = c.take<float>(2 * (size_t)g->N * d->heads);
    // the folded weights (the backward needs them too: formed again there they cost a launch of 6 to 12 us)
    const size_t fdd = hgt_folded(g, d) ? (size_t)g->R * d->d_out * d->d_out : 0;
    s->Wf_att = c.rows(fdd, h); s->Wf_msg = c.rows(fdd, h);
    return c.off;
}
size_t carve_hgt_fwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, void* base, HgtFwdWs* w) {
    Carver c(base);
    const size_t rdd = (size_t)g->R * d->d_out * d->d_out, fdd = hgt_folded(g, d) ? rdd : 0;
    w->Wbd_att = c.take<float>(rdd - fdd); w->Wbd_msg = c.take<float>(rdd - fdd);
    w->part_ms = c.take<float>(2 * (size_t)g->dst_items.num_partials * d->heads);
    w->partial = c.take<float>((size_t)g->dst_items.num_partials * d->d_out);
    return c.off;
}
size_t carve_hgt_bwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* d, void* base, HgtBwdWs* w) {
    Carver c(base);
    const bool h = rows_bf16(d);
    const bool fold = hgt_folded(g, d);
    const size_t D = d->d_out, rdd = (size_t)g->R * D * D, nd = (size_t)g->N * D, pd = (size_t)g->P * D;
    w->Wbd_att = c.take<float>(fold ? 0 : rdd); w->Wbd_msg = c.take<float>(fold ? 0 : rdd);
    w->dWbd_att = c.take<float>(fold ? 0 : rdd); w->dWbd_msg = c.take<float>(fold ? 0 : rdd);
    w->dWf_att = c.take<float>(fold ? rdd : 0); w->dWf_msg = c.take<float>(fold ? rdd : 0);
    w->dZ = c.rows(nd, h); w->adl = c.take<float>(2 * (size_t)g->E * d->heads);
    w->dKM = c.rows(2 * pd, h); w->dQ = c.rows(nd, h);
    w->dKp = c.rows(pd, h); w->dVp = c.rows(h && fold ? 0 : pd, h);     // folded, bf16 rows: dKp holds the sum of both
    w->dK = c.rows(fold ? 0 : nd, h); w->dV = c.rows(fold ? 0 : nd, h);
    w->dXk = c.take<float>(h || fold ? 0 : nd); w->dXq = c.take<float>((h && !fold) || hgt_pairs_with_query(g, d) ? 0 : nd); w->dXv = c.take<float>(h || fold ? 0 : nd);
    // shares of the weight gradients, which one launch adds: output, query (and unfolded value) linears; both pair linears
    const bool jobs = hgt_bwd_jobs(g, d);
    const size_t nodes = std::max(tl_bwd_scratch(h, node_chunks(g, d->d_out), d->d_in, d->d_out), jobs ? typed_linear_bwd_scratch_floats(D, D, g->node_tiles_hgt) : 0);
    const size_t query = std::max(nodes, hgt_pairs_with_query(g, d) ? (size_t)D * D * g->node_tiles_sum.num_slots : 0);
    const size_t pairs = std::max(tl_bwd_scratch(h, pair_chunks(g, d->d_out), d->d_in, d->d_out), jobs ? typed_linear_bwd_scratch_floats(D, D, g->pair_tiles_hgt) : 0);
    w->node_part[0] = c.take<float>(nodes); w->node_part[1] = c.take<float>(query); w->node_part[2] = c.take<float>(fold ? 0 : nodes);
    w->pair_part[0] = c.take<float>(pairs); w->pair_part[1] = c.take<float>(h && fold ? 0 : pairs);
    w->partial = c.take<float>(std::max(2 * (size_t)g->pair_items.num_partials, (size_t)g->dst_items.num_partials) * D);
    const bool acc = grads_accumulate(d);
    const size_t dh = D / d->heads;
    for (int i = 0; i < 4; ++i) w->acc_node[i] = acc ? c.take<float>((size_t)g->T * D * D) : nullptr;
    for (int i = 0; i < 2; ++i) w->acc_rel[i] = acc ? c.take<float>((size_t)g->R * d->heads * dh * dh) : nullptr;
    w->acc_mu = acc ? c.take<float>((size_t)g->R * d->heads) : nullptr;
    return c.off;
}

// Staging sizes: room for every tensor argument an entry point may widen (an upper bound at width 128,
// where most bf16 arguments are consumed as they are).
size_t stage_bytes(const rgnn_graph_t* g, int layer, const rgnn_layer_desc_t* d, bool bwd) {
    Bf16Stage s(nullptr, 0, d->dtype == RGNN_BF16, nullptr);
    const size_t N = g->N, R = g->R, T = g->T, di = d->d_in, dz = d->d_out;
    s.reserve(N * di);                                   // X
    if (layer == RGNN_LAYER_RGCN) { s.reserve(R * di * dz); s.reserve(di * dz); }
    if (layer == RGNN_LAYER_RGAT) { s.reserve(R * di * dz); s.reserve(R * dz); s.reserve(R * dz); }
    if (layer == RGNN_LAYER_HGT) {
        const size_t dh = dz / d->heads;
        for (int i = 0; i < 4; ++i) s.reserve(T * dz * dz);
        s.reserve(R * d->heads * dh * dh); s.reserve(R * d->heads * dh * dh); s.reserve(R * d->heads);
    }
    if (bwd) s.reserve(N * dz);                          // dOut
    return s.c.off;
}

// Inference calls (saved == NULL): the tensors a backward call would need are still intermediates of
// the forward, and live behind the forward scratch and the staging area in the workspace.
void* saved_or_scratch(const rgnn_graph_t* g, int layer, const rgnn_layer_desc_t* d, void* saved, void* workspace,
                       size_t fwd_carved) {
    if (saved) return saved;
    return static_cast<char*>(workspace) + align_up(fwd_carved + stage_bytes(g, layer, d, false));
}

// Forward typed linear  Y[g(i)] / Y[i] = A[g(i)] W[seg].  In bf16 mode it runs on the bf16 matrix
// cores: an operand whose bf16 form exists (A16 / W16) is used as is, an fp32-only one is split.
// y16: the output rows are stored as bf16 (width 128 only).
// Chunking: the bf16 kernel with fp32 results and the weight in bf16 does best on many short chunks; when the weight has to be
// split, and in the fp32 kernels, loading a segment's weight costs more and one resident round of long chunks wins.
// d_in (fp32 kernels only): width of the input rows when it differs from the output width d.
// y_stride: the output rows are y_stride * d elements apart.
rgnn_status_t tl_fwd(bool bf16, const Chunkings& tiles, int d, const float* A32,
                     const void* A16, const int32_t* gather, int scatter, const float* W32, const void* W16, void* Y,
                     bool y16, const char* label, hipStream_t st, int d_in = 0, int y_stride = 1, bool sign_matters = false) {
    if (d_in == 0) d_in = d;
    if (bf16) {
        if (d_in != d) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear on the bf16 matrix cores: equal widths only");
        if (A16 && W16 && y16 && gather && y_stride == 1) return typed_linear_fwd_bf16({tiles.cu2, A16, gather, scatter, W16, nullptr, Y, label}, st);
        TypedLinearBf16Args a{};
        a.tiles = W16 ? tiles.many : tiles.wide; a.A = A16 ? A16 : A32; a.a_bf16 = A16 != nullptr; a.gather = gather; a.scatter_out = scatter;
        a.W = W16 ? W16 : W32; a.w_bf16 = W16 != nullptr; a.Y = Y; a.y_bf16 = y16; a.label = label;
        a.y_stride = y_stride;
        return typed_linear_bf16(d, a, st);
    }
    TypedLinearArgs a{};
    a.tiles = tiles.f32; a.X = A32; a.gather = gather; a.W = W32; a.Y = static_cast<float*>(Y); a.scatter_out = scatter;
    a.label = label; a.y_stride = y_stride; a.sign_matters = sign_matters;
    return typed_linear_fwd(d_in, d, a, st);
}

// Backward typed linear: dXrow = dY W^T (rows through `gather` on both sides when `both_gathered`),
// dW = sum X^T dY.
//   rows16 (bf16 rows, width 128): X and dY are bf16; one kernel on the bf16 matrix cores (the weight as is when its
//     bf16 form W16 exists, split into two planes otherwise) and the slot reduction.  dXrow is stored as bf16 (dx16) or fp32.
//   otherwise: the fused fp32 kernel on fp32 X, W, dY.
//   dx_acc: dXrow += (fp32 dXrow, rows16)
//   dy_stride: the rows of dY are dy_stride * d elements apart (dY not gathered)
//   ysel / y_alt (dY not gathered): row i of dY is dY[ysel[i]], or y_alt[ysel[i] & 0x7FFFFFFF] when the
//     top bit of ysel[i] is set; with yscale it is also multiplied by yscale[i]
rgnn_status_t tl_bwd(bool rows16, const Chunkings& tiles, int d, const void* X,
                     const int32_t* gather, int both_gathered, const float* W32, const void* W16, const void* dY,
                     void* dXrow, bool dx16, float* dW, float* part, const char* label, hipStream_t st,
                     bool dx_acc = false, const int32_t* ysel = nullptr, const void* y_alt = nullptr,
                     const float* yscale = nullptr, int d_in = 0, int dy_stride = 1, ShareSums* sums = nullptr) {
    if (d_in == 0) d_in = d;
    if (rows16 && d_in != d) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear backward on the bf16 matrix cores: equal widths only");
    if (ysel && both_gathered) RGNN_FAIL(RGNN_EUNSUPPORTED, "row selector: ungathered dY only");
    if (rows16) {
        TypedLinearBwdBf16Args a{};
        a.tiles = W16 ? tiles.cu2 : tiles.cu1; a.X = X; a.gather = gather; a.both_gathered = both_gathered;
        a.W = W16 ? W16 : W32; a.w_bf16 = W16 != nullptr; a.dY = dY; a.dy_stride = dy_stride; a.dXrow = dXrow; a.dx_f32 = !dx16;
        a.accumulate = dx_acc; a.dW = dW; a.part = part; a.label = label; a.ysel = ysel; a.dY_alt = y_alt; a.yscale = yscale; a.sums = sums;
        return typed_linear_bwd_bf16(d, a, st);
    }
    if (dx_acc) RGNN_FAIL(RGNN_EUNSUPPORTED, "accumulating input gradient needs bf16 rows");
    TypedLinearBwdArgs b{};
    b.tiles = tiles.f32_bwd; b.X = static_cast<const float*>(X); b.gather = gather; b.W = W32; b.dY = static_cast<const float*>(dY);
    b.dy_gathered = both_gathered; b.dXrow = static_cast<float*>(dXrow); b.scatter_dx = both_gathered; b.dW = dW;
    b.part = part; b.label = label; b.dy_stride = dy_stride;
    b.ysel = ysel; b.dY_alt = static_cast<const float*>(y_alt); b.yscale = yscale; b.sums = sums;
    return typed_linear_bwd(d_in, d, b, st);
}
// A forward that keeps nothing (what fits the static scratch with rows per pair only takes those, with a workspace of the caller's too).
bool rgat_run_rows_infer(const rgnn_graph_t* g, const rgnn_layer_desc_t* d) {
    if (!rgat_run_rows(g, d) || !sched_rgat_run_rows_infer(g->R, g->E, d->d_out)) return false;
    RgatFwdWs fw; RgatSaved ps; RgatRunSaved rs;
    const size_t f = align_up(carve_rgat_fwd(g, d, nullptr, &fw) + stage_bytes(g, RGNN_LAYER_RGAT, d, false));
    const size_t most = RGNN_STATIC_SCRATCH_BYTES;
    return f + carve_rgat_run_saved(g, d, nullptr, &rs, false) <= most || f + carve_rgat_saved(g, d, nullptr, &ps) > most;
}
}  // namespace

extern "C" rgnn_status_t rgnn_workspace_bytes(const rgnn_graph_t* g, int32_t layer, const rgnn_layer_desc_t* desc,
                                              size_t* fwd_workspace, size_t* bwd_workspace, size_t* saved) {
    if (layer != RGNN_LAYER_RGCN && layer != RGNN_LAYER_RGAT && layer != RGNN_LAYER_HGT)
        RGNN_FAIL(RGNN_EINVAL, "unknown layer %d", layer);
    RGNN_TRY(check_desc(g, desc, layer));
    size_t f = 0, b = 0, s = 0;
    if (layer == RGNN_LAYER_RGAT) {
        RgatFwdWs fw; RgatBwdWs bw; RgatSaved sv;
        f = carve_rgat_fwd(g, desc, nullptr, &fw);
        RgatRunBwdWs rb; RgatRunSaved rs;
        b = rgat_run_rows(g, desc) ? carve_rgat_run_bwd(g, desc, nullptr, &rb) : carve_rgat_bwd(g, desc, nullptr, &bw);
        s = carve_rgat_saved(g, desc, nullptr, &sv);
        if (rgat_keeps_runs(g, desc))
            for (bool kept : {true, false}) s = std::max(s, carve_rgat_run_saved(g, desc, nullptr, &rs, kept));
    } else if (layer == RGNN_LAYER_RGCN) {
        RgcnFwdWs fw; RgcnBwdWs bw;
        float* A;
        for (bool loop : {false, true}) {
            f = std::max(f, carve_rgcn_fwd(g, desc, loop, nullptr, &fw));
            b = std::max(b, carve_rgcn_bwd(g, desc, loop, nullptr, &bw));
            s = std::max(s, carve_rgcn_saved(g, desc, loop, nullptr, &A));
        }
    } else {
        HgtFwdWs fw; HgtBwdWs bw; HgtSaved sv;
        f = carve_hgt_fwd(g, desc, nullptr, &fw);
        b = carve_hgt_bwd(g, desc, nullptr, &bw);
        s = carve_hgt_saved(g, desc, nullptr, &sv);
    }
    f += stage_bytes(g, layer, desc, false);
    b += stage_bytes(g, layer, desc, true);
    if (fwd_workspace) *fwd_workspace = f;
    if (bwd_workspace) *bwd_workspace = b;
    if (saved) *saved = s;
    return RGNN_OK;
}

extern "C" rgnn_status_t rgnn_schedule(const rgnn_graph_t* g, int32_t layer, const rgnn_layer_desc_t* desc, rgnn_schedule_t* out) {
    if (layer != RGNN_LAYER_RGCN && layer != RGNN_LAYER_RGAT && layer != RGNN_LAYER_HGT)
        RGNN_FAIL(RGNN_EINVAL, "unknown layer %d", layer);
    RGNN_TRY(check_desc(g, desc, layer));
    if (!out) RGNN_FAIL(RGNN_EINVAL, "out is NULL");
    ScheduleIn in;
    in.layer = layer; in.dtype = desc->dtype; in.d = desc->d_out; in.heads = layer == RGNN_LAYER_RGCN ? 1 : desc->heads;
    in.flags = desc->flags; in.R = g->R; in.edges = g->E; in.rel_src_tied = g->rel_src_tied;
    const Chunkings pc = pair_chunks(g, desc->d_out);
    in.item_len = item_cut(g->E); in.tile_chunks = pc.many->num_chunks;
    const bool rows16 = layer != RGNN_LAYER_RGAT && rows_bf16(desc);
    in.wide_chunks = (rows16 ? (layer == RGNN_LAYER_RGCN ? pc.cu2 : pc.cu1)
                             : layer == RGNN_LAYER_HGT && hgt_bwd_jobs(g, desc) ? hgt_pair_list(g, desc->d_out) : pc.f32_bwd)->num_chunks;
    in.dst = {g->dst_items.num_single, g->dst_items.num_short};
    in.pair = {g->pair_items.num_single, g->pair_items.num_short};
    in.pair_multi = {g->pair_items_multi.num_single, g->pair_items_multi.num_short};
    *out = pick_schedule(in);
    return RGNN_OK;
}

// =========================================================================== RGCN

// A[m] = sum over the edges of the m-th run with several edges of X[src_e] / c, or of X[src_e]
static rgnn_status_t rgcn_run_inputs(const rgnn_graph_t* g, const rgnn_layer_desc_t* desc, const float* X, float* A, float* partial, hipStream_t st) {
    const float* coef = desc->norm == RGNN_NORM_IN_DEGREE_PER_REL ? g->in_invc : nullptr;
    return gather_sum(g->multi_run_items, desc->d_in, nullptr, g->idx[RGNN_IDX_IN_SRC], 0, coef, 1, 0, X, A, partial, st, 1, "run_inputs", "run_inputs.combine");
}

extern "C" rgnn_status_t rgnn_rgcn_fwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* desc, const void* X,
                                       const void* W, const void* W0, void* out, void* saved, void* workspace,
                                       void* stream) {
    RGNN_TRY(check_desc(g, desc, RGNN_LAYER_RGCN));
    ScheduleFlagsScope sched_scope(desc->flags);
    if (missing(g, X) || !W || missing(g, out)) RGNN_FAIL(RGNN_EINVAL, "X, W or out is NULL");
    if (!workspace) RGNN_FAIL(RGNN_EWORKSPACE, "workspace is NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int D = desc->d_out;
    RgcnFwdWs w;
    const bool bf16 = desc->dtype == RGNN_BF16, h = rows_bf16(desc), relu = desc->activation == RGNN_ACT_RELU;
    const void* X16 = bf16 ? X : nullptr;
    const void* W16 = bf16 ? W : nullptr;
    Bf16Stage stg(workspace, carve_rgcn_fwd(g, desc, W0 != nullptr, workspace, &w), bf16, st);
    // fp32 copies for the fp32 kernels: everything below width 128, only the self-loop operands at 128
    const float* X32 = (!h || W0) ? stg.in(X, (size_t)g->N * desc->d_in) : nullptr;
    const float* W32 = !h ? stg.in(W, (size_t)g->R * desc->d_in * D) : nullptr;
    const float* W032 = stg.in(W0, (size_t)desc->d_in * D);
    RGNN_TRY(stg.status);
    // What the backward reads is left in `saved` whatever the flags: the backward cannot tell.
    const bool runs = rgcn_run_rows(g, desc, W0) && (saved || sched_run_rows_infer(g->E, D));
    float* A = w.A;
    if (saved && rgcn_keeps_sums(g, desc, W0)) {
        (void)carve_rgcn_saved(g, desc, W0, saved, &A);
        RGNN_TRY(rgcn_run_inputs(g, desc, X32, A, w.partial, st));
    }
    // (one launch: rows of out are written while others of X are still read, so an out that shares memory with X goes to the
    // general plan, which has read X by then unless there is a self-loop)
    if (!overlap(X, (size_t)g->N * desc->d_in * sizeof(float), out, (size_t)g->N * D * sizeof(float)) &&
        rgcn_small(g, desc, W0, desc->flags))
        return rgcn_small_fwd(g, desc->d_in, D, X32, W32, W032, desc->norm == RGNN_NORM_IN_DEGREE_PER_REL, relu, static_cast<float*>(out), st);
    if (runs) {
        // The sum over a run's edges comes before the product: a row of messages per run, not per pair, and a run with one edge reads its
        // source's row directly.
        if (!saved) RGNN_TRY(rgcn_run_inputs(g, desc, X32, A, w.partial, st));
        TypedLinearArgs a{};
        a.tiles = run_chunks(g, D).f32; a.X = X32; a.X2 = A; a.gather = g->row_in; a.to = g->row_run; a.W = W32; a.Y = static_cast<float*>(w.Hs); a.sign_matters = 1;
        RGNN_TRY(typed_linear_fwd(desc->d_in, D, a, st));
        RGNN_TRY(gather_sum(g->dstrun_items, D, nullptr, nullptr, 0, nullptr, 1, 0, w.Hs, out, w.partial, st, 0, "aggregate_fwd", "aggregate_fwd.combine"));
    } else {
        // 1. compact messages: Hs[p] = X[pair_src[p]] W[rel(p)]
        RGNN_TRY(tl_fwd(bf16, pair_chunks(g, D), D, X32, X16, g->idx[RGNN_IDX_PAIR_SRC], 0, W32, W16, w.Hs, h, "typed_linear_fwd", st,
                        desc->d_in, 1, true));
        // 2. out[v] = sum_e (1/c) Hs[pair_e]
        const float* coef = desc->norm == RGNN_NORM_IN_DEGREE_PER_REL ? g->in_invc : nullptr;
        RGNN_TRY(gather_sum(g->dst_items, D, nullptr, g->idx[RGNN_IDX_IN_PAIR], 0, coef, 1, 0, w.Hs, out, w.partial, st, 0,
                            "aggregate_fwd", "aggregate_fwd.combine", 1, h, 0));
    }
    // 3. self-loop: out += X W0, and the activation on the way out (a pass of its own over out took 16.5 us at 120k
    //    nodes of width 64; without a self-loop it still is one)
    if (W0) {
        TypedLinearArgs s{};
        s.tiles = all_chunks(g, D); s.X = X32; s.W = W032;
        s.Y = static_cast<float*>(out); s.accumulate = 1; s.relu = relu; s.sign_matters = 1; s.label = "self_loop_fwd";
        RGNN_TRY(typed_linear_fwd(desc->d_in, D, s, st));
    }
    if (relu && !W0) RGNN_TRY(relu_inplace((size_t)g->N * D, static_cast<float*>(out), st));
    return RGNN_OK;
}

extern "C" rgnn_status_t rgnn_rgcn_bwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* desc, const void* X,
                                       const void* W, const void* W0, const void* out, const void* saved,
                                       const void* dOut, void* dX, void* dW, void* dW0, void* workspace,
                                       void* stream) {
    RGNN_TRY(check_desc(g, desc, RGNN_LAYER_RGCN));
    ScheduleFlagsScope sched_scope(desc->flags);
    if (missing(g, X) || !W || missing(g, dOut) || missing(g, dX) || !dW) RGNN_FAIL(RGNN_EINVAL, "a required tensor pointer is NULL");
    if (W0 && !dW0) RGNN_FAIL(RGNN_EINVAL, "dW0 is NULL but W0 is given");
    if (desc->activation != RGNN_ACT_NONE && missing(g, out)) RGNN_FAIL(RGNN_EINVAL, "out is needed for the activation's gradient");
    if (!workspace) RGNN_FAIL(RGNN_EWORKSPACE, "workspace is NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int D = desc->d_out, K = desc->d_in;
    RgcnBwdWs w;
    const bool bf16 = desc->dtype == RGNN_BF16, h = rows_bf16(desc), relu = desc->activation == RGNN_ACT_RELU;
    const void* W16 = bf16 ? W : nullptr;
    Bf16Stage stg(workspace, carve_rgcn_bwd(g, desc, W0 != nullptr, workspace, &w), bf16, st);
    const float* X32 = (!h || W0) ? stg.in(X, (size_t)g->N * K) : nullptr;
    const float* W32 = !h ? stg.in(W, (size_t)g->R * K * D) : nullptr;
    const float* W032 = stg.in(W0, (size_t)K * D);
    const float* dO32 = !h || (W0 && !relu) ? stg.in(dOut, (size_t)g->N * D) : nullptr;   // (h, W0 and relu: dPre32 instead)
    RGNN_TRY(stg.status);
    const bool acc = grads_accumulate(desc);
    GradAcc ga;
    dW = ga.route(w.acc_dW, dW, (size_t)g->R * K * D);
    dW0 = ga.route(w.acc_dW0, dW0, (size_t)K * D);
    // gradient before the activation, in the storage the traversal reads (dPre) and, where an fp32
    // kernel needs it, in fp32 (dPre32)
    const void* dPre = h ? dOut : dO32;
    const float* dPre32 = dO32;
    if (relu) {
        const bool both = h && W0;
        RGNN_TRY(relu_grad((size_t)g->N * D, static_cast<const float*>(out), dPre, w.dPre, st, h, both ? w.dPre32 : nullptr));
        dPre = w.dPre;
        dPre32 = both ? w.dPre32 : h ? nullptr : static_cast<const float*>(w.dPre);
    }
    const bool runs = rgcn_run_rows(g, desc, W0);
    const float* A = w.A;
    if (runs && saved) {
        float* kept = nullptr;
        (void)carve_rgcn_saved(g, desc, W0, const_cast<void*>(saved), &kept);
        A = kept;
    } else if (runs) {
        RGNN_TRY(rgcn_run_inputs(g, desc, X32, w.A, w.partial, st));
    }
    // 1. dHs[p] = sum_{e in out(p)} (1/c_e) dPre[dst_e]     (rows per run: the row of run q is dPre[dst_q])
    const float* coef = desc->norm == RGNN_NORM_IN_DEGREE_PER_REL ? g->in_invc : nullptr;
    //    (coefficients from the pair-major copy, so no per-edge indirection is left)
    const float* ocoef = coef ? g->out_invc : nullptr;
    //    With the row selector the row of a pair with a single edge is not written per pair: the typed-linear backward
    //    reads dPre[dst_e] instead and multiplies it by 1/c_e on the way in.
    const bool sel = sched_row_select(RGNN_LAYER_RGCN, desc->dtype, D, 1, g->R, g->E, g->pair_items.num_single, desc->flags);
    const int32_t* ysel = sel ? g->pair_ysel : nullptr;
    const void* y_alt = sel ? dPre : nullptr;
    const float* yscale = sel && coef ? g->pair_scale : nullptr;
    if (!runs)
        RGNN_TRY(gather_sum(sel ? g->pair_items_multi : g->pair_items, D, nullptr, g->idx[RGNN_IDX_OUT_DST], 0, ocoef, 1, 0, dPre, w.G,
                            w.partial, st, 1, "aggregate_bwd_pair", "aggregate_bwd_pair.combine", 1, h, h));
    // 2. per pair dXp = dHs W^T; dW[r] = sum X^T dHs (its shares are added with those of the self-loop)
    ShareSums sums;
    // 3. self-loop: dX0 = dPre W0^T, dW0 = X^T dPre
    TypedLinearBwdArgs s{};
    s.tiles = &g->all_tiles_cu1; s.X = X32; s.W = W032; s.dY = dPre32;
    s.dXrow = w.dX0; s.dW = static_cast<float*>(dW0); s.part = w.loop_part; s.label = "self_loop_bwd"; s.sums = &sums;
    TypedLinearBwdArgs b{};
    b.X = X32; b.W = W32; b.dXrow = static_cast<float*>(w.dXp); b.dW = static_cast<float*>(dW); b.part = w.tl_part; b.sums = &sums;
    if (runs) {
        b.X2 = A; b.gather = g->row_in; b.dY = static_cast<const float*>(dPre); b.ysel = g->row_dst;
    } else {
        b.gather = g->idx[RGNN_IDX_PAIR_SRC]; b.dY = static_cast<const float*>(w.G); b.ysel = ysel; b.dY_alt = static_cast<const float*>(y_alt); b.yscale = yscale;
    }
    if (W0 && rgcn_loop_bwd(g, desc)) {
        b.tiles = runs ? &g->run_tiles_loop : &g->pair_tiles_loop;
        s.tiles = runs ? &g->all_tiles_run_loop : &g->all_tiles_loop;
        RGNN_TRY(typed_linear_bwd_loop(K, D, b, s, st));
    } else if (runs) {
        b.tiles = run_chunks(g, D).f32_bwd;
        RGNN_TRY(typed_linear_bwd(K, D, b, st));
        if (W0) RGNN_TRY(typed_linear_bwd(K, D, s, st));
    } else {
        RGNN_TRY(tl_bwd(h, pair_chunks(g, D), D, h ? X : static_cast<const void*>(X32), g->idx[RGNN_IDX_PAIR_SRC], 0, W32, W16, w.G,
                        w.dXp, h, static_cast<float*>(dW), w.tl_part, "typed_linear_bwd", st, false, ysel, y_alt, yscale, K, 1, &sums));
        if (W0) RGNN_TRY(typed_linear_bwd(K, D, s, st));
    }
    RGNN_TRY(sums.launch(st));
    // 4. dX[u] = sum over u's pairs of dXp (+ dX0[u]) (+ what dX holds, when gradients accumulate)
    const float* extra = W0 ? w.dX0 : nullptr;
    if (acc && W0) RGNN_TRY(add_into((size_t)g->N * K, static_cast<const float*>(dX), w.dX0, st));
    else if (acc) extra = static_cast<const float*>(dX);
    if (runs)      // over u's edges: the row of the edge's run, times 1/c
        RGNN_TRY(gather_sum(g->src_items, K, nullptr, g->src_row, 0, coef ? g->src_invc : nullptr, 1, 0, w.dXp, dX, w.partial, st, 3, "node_grad_sum",
                            "node_grad_sum.combine", 1, 0, 0, nullptr, extra));
    else
        RGNN_TRY(node_grad_sum(g, K, w.dXp, nullptr, nullptr, extra, dX, st, h, 0));
    return ga.flush(st);
}

// =========================================================================== RGAT

namespace {

// The library's own scratch for rgnn_rgat_fwd_static: device memory inside the code object, one copy per GPU,
// held until the process ends.  In host code the array's name is only a handle for hipGetSymbolAddress; the
// device address it yields (per device) is what kernels and carve-outs use.
static __device__ __align__(256) unsigned char scratch[RGNN_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

}  // namespace

namespace rgnn {
// Address of the static scratch array on the current device; looked up once per device and kept.
rgnn_status_t static_scratch(void** p) {
    int dev = 0;
    RGNN_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) RGNN_FAIL(RGNN_EUNSUPPORTED, "device ordinal %d is beyond the %d the library tracks", dev, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        RGNN_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) RGNN_FAIL(RGNN_EHIP, "hipGetSymbolAddress returned a null address for the static scratch");
        g_scratch_ptr[dev] = ptr;
    }
    *p = g_scratch_ptr[dev];
    return RGNN_OK;
}
}  // namespace rgnn

static rgnn_status_t rgat_fwd_impl(const rgnn_graph_t* g, const rgnn_layer_desc_t* desc, const void* X, const void* W, const void* w_s,
                                   const void* w_t, void* out, void* saved, void* workspace, void* stream);

extern "C" rgnn_status_t rgnn_rgat_fwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* desc, const void* X,
                                       const void* W, const void* w_s, const void* w_t, void* out, void* saved,
                                       void* workspace, void* stream) {
    return rgat_fwd_impl(g, desc, X, W, w_s, w_t, out, saved, workspace, stream);
}

extern "C" rgnn_status_t rgnn_rgat_fwd_static(const rgnn_graph_t* g, const rgnn_layer_desc_t* desc, const void* X,
                                              const void* W, const void* w_s, const void* w_t, void* out, void* saved,
                                              void* stream) {
    size_t need = 0;
    RGNN_TRY(rgnn_workspace_bytes(g, RGNN_LAYER_RGAT, desc, &need, nullptr, nullptr));
    if (!saved) {                                // inference: the would-be saved tensors are scratch too
        RgatSaved ps; RgatRunSaved rs;
        need = align_up(need) + (rgat_run_rows_infer(g, desc) ? carve_rgat_run_saved(g, desc, nullptr, &rs, false) : carve_rgat_saved(g, desc, nullptr, &ps));
    }
    if (need > (size_t)RGNN_STATIC_SCRATCH_BYTES)
        RGNN_FAIL(RGNN_EWORKSPACE, "rgnn_rgat_fwd_static: this call needs %zu bytes of scratch, the static buffer holds %zu",
                  need, (size_t)RGNN_STATIC_SCRATCH_BYTES);
    void* ws = nullptr;
    RGNN_TRY(static_scratch(&ws));
    return rgat_fwd_impl(g, desc, X, W, w_s, w_t, out, saved, ws, stream);
}

static rgnn_status_t rgat_pair_fwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* desc, const float* Xf, const float* Wf, const float* w_s,
                                   const float* w_t, void* out, void* saved, const RgatFwdWs& w, hipStream_t st);

static rgnn_status_t rgat_fwd_impl(const rgnn_graph_t* g, const rgnn_layer_desc_t* desc, const void* X, const void* W, const void* w_s,
                                   const void* w_t, void* out, void* saved, void* workspace, void* stream) {
    RGNN_TRY(check_desc(g, desc, RGNN_LAYER_RGAT));
    ScheduleFlagsScope sched_scope(desc->flags);
    if (missing(g, X) || !W || !w_s || !w_t || missing(g, out)) RGNN_FAIL(RGNN_EINVAL, "a required tensor pointer is NULL");
    if (!workspace) RGNN_FAIL(RGNN_EWORKSPACE, "workspace is NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int D = desc->d_out, K = desc->d_in;
    RgatFwdWs w; RgatRunSaved rs;
    const size_t carved = carve_rgat_fwd(g, desc, workspace, &w);
    const bool kept = saved && rgat_keeps_runs(g, desc);
    saved = saved_or_scratch(g, RGNN_LAYER_RGAT, desc, saved, workspace, carved);
    Bf16Stage stg(workspace, carved, desc->dtype == RGNN_BF16, st);
    X = stg.in(X, (size_t)g->N * K);
    W = stg.in(W, (size_t)g->R * K * D);
    w_s = stg.in(w_s, (size_t)g->R * D);
    w_t = stg.in(w_t, (size_t)g->R * D);
    RGNN_TRY(stg.status);
    const float *Xf = static_cast<const float*>(X), *Wf = static_cast<const float*>(W), *ws = static_cast<const float*>(w_s), *wt = static_cast<const float*>(w_t);
    // (with an out that shares memory with X, what is kept cannot be formed behind the rows per pair: then no flag brings those back)
    const bool runs = kept ? rgat_run_rows(g, desc) || overlap(Xf, (size_t)g->N * K * sizeof(float), out, (size_t)g->N * D * sizeof(float))
                           : rgat_run_rows_infer(g, desc);
    if (runs || kept) carve_rgat_run_saved(g, desc, saved, &rs, kept);
    if (runs) {
        // 1. wsp = W w_s, wtp = W w_t, and the destination halves of the logits
        RGNN_TRY(fold_weight(fold_args(g->R, K, D, 1, Wf, ws, rs.wsp, wt, rs.wtp), st));
        RGNN_TRY(rgat_run_logit(g, K, Xf, rs.wtp, rs.s_dst, st));
        // 2. the inputs of the runs with several edges, weighted within the run;  3. Y = A W, a run with one edge reading its source's row
        RGNN_TRY(rgat_run_inputs(g, K, Xf, rs.wsp, rs.s_dst, desc->slope, rs.A, rs.lq, rs.partial, rs.part_ms, st));
        TypedLinearArgs a{};
        a.tiles = run_chunks(g, D).f32; a.X = Xf; a.X2 = rs.A; a.gather = g->row_in; a.to = g->row_run; a.W = Wf; a.Y = rs.Y; a.sign_matters = 1;
        RGNN_TRY(typed_linear_fwd(K, D, a, st));
        // 4. per destination over its runs: softmax and weighted sum
        return rgat_run_aggregate(g, D, rs.Y, ws, rs.s_dst, desc->slope, rs.lq, static_cast<float*>(out), rs.ms, w.partial, w.part_ms, st);
    }
    RGNN_TRY(rgat_pair_fwd(g, desc, Xf, Wf, ws, wt, out, saved, w, st));
    if (!kept) return RGNN_OK;
    // what rows per run need beside s_dst and (m, s), in the place of Hs and behind
    RGNN_TRY(fold_weight(fold_args(g->R, K, D, 1, Wf, ws, rs.wsp, wt, rs.wtp), st));
    RGNN_TRY(rgat_run_inputs(g, K, Xf, rs.wsp, rs.s_dst, desc->slope, rs.A, rs.lq, rs.partial, rs.part_ms, st));
    return rgat_single_logits(g, K, Xf, rs.wsp, rs.s_dst, desc->slope, rs.lq, st);
}

// Rows per pair; X .. w_t in fp32.
static rgnn_status_t rgat_pair_fwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* desc, const float* Xf, const float* Wf, const float* w_s,
                                   const float* w_t, void* out, void* saved, const RgatFwdWs& w, hipStream_t st) {
    const int D = desc->d_out, K = desc->d_in;
    RgatSaved sv;
    carve_rgat_saved(g, desc, saved, &sv);
    const bool fused = rgat_fused(desc);
    // 1. compact messages: Hs[p] = X[pair_src[p]] W[r]
    //    (the comparison schedules also take the source half of the logit per pair, s_src[p] = Hs[p] . w_s[r])
    TypedLinearArgs a{};
    a.sign_matters = 1;
    a.tiles = pair_chunks(g, D).f32; a.X = Xf; a.gather = g->idx[RGNN_IDX_PAIR_SRC]; a.W = Wf; a.Y = sv.Hs;
    if (!fused) { a.vec = w_s; a.s_out = w.s_src; }
    const int H = desc->heads;
    const FoldArgs fold = fold_args(g->R, K, D, H, Wf, w_t, w.wtp);      // step 2; in the same launch if there is one
    // At width 128 the product's LDS leaves a compute unit one workgroup of folds at a time: with many relations they are faster in a
    // launch of their own, unless uneven chunks leave compute units idle.  Forward, us, shared / apart, equal frequencies: 200 relations
    // 76 / 76 at 100k edges, 800 111 / 104, 2000 192 / 152, 566 / 538 at 1M; Zipf 1.1: 400 55 / 49 at 10k, 97 / 102 at 100k, 2000 803 / 824 at 1M.
    // (With heads the folds read W by columns and are slow alone: 2000 relations 234 / 392 at 100k.)
    const bool lone_folds = K == 128 && H == 1 && fold.blocks > 4 * g->num_cus && !a.tiles->uneven();
    const bool with_fold = fused && a.tiles->num_tiles > 0 && fold_rides(fold) && !lone_folds;
    if (with_fold) a.fold = &fold;
    RGNN_TRY(typed_linear_fwd(K, D, a, st));
    // 2. destination half, once per (dst, rel) run, reordered: s_dst[q] = X[dst] . (W[r] w_t[r])  (per head: the head's columns)
    if (!with_fold) RGNN_TRY(fold_weight(fold, st));
    RGNN_TRY(run_logit(g, K, H, Xf, w.wtp, sv.s_dst, st));
    if (!fused) {
        // 3'. edge softmax in a pass of its own (one attention weight per edge, and (max, sum) per destination for the
        //     backward call), then the weighted sum: by the destination-segment walk, or edge by edge with atomic adds
        RGNN_TRY(edge_softmax(g, w.s_src, sv.s_dst, desc->slope, w.att, w.part_m, w.part_s, st, sv.ms));
        if (rgat_edge_parallel(desc)) return aggregate_edge_parallel(g, D, w.att, sv.Hs, static_cast<float*>(out), st);
        return gather_sum(g->dst_items, D, nullptr, g->idx[RGNN_IDX_IN_PAIR], 0, w.att, 1, 1, sv.Hs, static_cast<float*>(out),
                          w.partial, st, 0, "aggregate_fwd", "aggregate_fwd.combine");
    }
    // 3. one walk per destination: logit from the gathered row, running-maximum softmax, weighted sum
    return rgat_aggregate_fwd(g, D, H, sv.Hs, w_s, sv.s_dst, desc->slope, static_cast<float*>(out), sv.ms, w.partial, w.part_ms, st);
}

// Rows per run; X .. dOut in fp32.
static rgnn_status_t rgat_run_bwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* desc, const float* X, const float* W, const float* w_s,
                                  const float* w_t, const void* saved, const float* dOut, float* dX, void* dW, void* dw_s, void* dw_t,
                                  const RgatRunBwdWs& w, hipStream_t st) {
    const int D = desc->d_out, K = desc->d_in;
    RgatRunSaved sv;
    carve_rgat_run_saved(g, desc, const_cast<void*>(saved), &sv, true);
    GradAcc ga;
    dW = ga.route(w.acc_dW, dW, (size_t)g->R * K * D);
    dw_s = ga.route(w.acc_dws, dw_s, (size_t)g->R * D);
    dw_t = ga.route(w.acc_dwt, dw_t, (size_t)g->R * D);
    ShareSums sums;
    auto pieces = [&](const ItemList& L, const float* partial, float* to) {
        return SumArgs{partial, L.split_row, L.split_ptr, to, (size_t)L.num_partials * K, (size_t)g->R * K, L.num_split, K, 1};
    };
    RGNN_TRY(rgat_run_weights(g, sv.ms, sv.lq, w.weight, st));
    // 1. dH[q] = dOut[dst_q] W[r]^T;  dW[r] = sum over r's runs of (weight A[q])^T dOut[dst_q];  rowdot = dH[q] . weight A[q]
    TypedLinearBwdArgs b{};
    b.tiles = run_chunks(g, D).f32_bwd; b.X = X; b.X2 = sv.A; b.gather = g->row_in; b.W = W; b.dY = dOut; b.ysel = g->row_dst; b.yscale = w.weight;
    b.rowdot = w.rowdot; b.num = g->row_run;
    b.dXrow = w.dH; b.dW = static_cast<float*>(dW); b.part = w.tl_part; b.sums = &sums;
    RGNN_TRY(typed_linear_bwd(K, D, b, st));
    // 2. what the edges of a run need
    RGNN_TRY(rgat_run_stat(g, desc->slope, w.rowdot, w.weight, sv.ms, sv.lq, sv.s_dst, w.stat, w.ds_dst, st));
    // 3. per source over its edges: dz, and dX without the destination halves
    //    (with a dX that shares memory with X, which step 4 reads, dz alone, and the walk again behind that)
    const bool in_place = overlap(X, (size_t)g->N * K * sizeof(float), dX, (size_t)g->N * K * sizeof(float));
    auto walk = [&](float* to) {
        return rgat_source_walk(g, K, X, w.dH, sv.wsp, w.stat, desc->slope, w.dz, to, grads_accumulate(desc), w.partial, st);
    };
    RGNN_TRY(walk(in_place ? nullptr : dX));
    // 4. sums of dz over the runs with several edges;  A[r] = sum over r's pairs of ds_src X[src], U[r] = sum over r's runs of ds_dst X[dst]
    RGNN_TRY(segment_scalar_sum((int)g->Q, g->idx[RGNN_IDX_RUN_PTR], g->long_runs, g->in_spos, w.dz, 1, 0, w.ds_dst, st, "ds_dst_sum", 2));
    RGNN_TRY(rgat_block_sums(g, K, X, w.dz, w.ds_src, w.ds_dst, w.A, w.a_partial, w.U, w.u_partial, st));
    if (in_place) RGNN_TRY(walk(dX));
    sums.pieces = pieces(g->pair_blocks, w.a_partial, w.A);
    sums.pieces2 = pieces(g->run_blocks, w.u_partial, w.U);
    RGNN_TRY(sums.launch(st));
    // 5. dX[v] += sum over v's runs of ds_dst[q] (W[r] w_t[r]);  dw_s = A W, dw_t = U W, dW += A^T (x) w_s + U^T (x) w_t
    const RgatFinish fin{g->R, K, D, 1, W, w_s, w_t, w.A, w.U, static_cast<float*>(dW), static_cast<float*>(dw_s), static_cast<float*>(dw_t), 0};
    RGNN_TRY(rgat_run_term(g, K, w.ds_dst, sv.wtp, dX, fin, st));
    return ga.flush(st);
}

extern "C" rgnn_status_t rgnn_rgat_bwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* desc, const void* X,
                                       const void* W, const void* w_s, const void* w_t, const void* out,
                                       const void* saved, const void* dOut, void* dX, void* dW, void* dw_s,
                                       void* dw_t, void* workspace, void* stream) {
    RGNN_TRY(check_desc(g, desc, RGNN_LAYER_RGAT));
    ScheduleFlagsScope sched_scope(desc->flags);
    if (missing(g, X) || !W || !w_s || !w_t || missing(g, out) || missing(g, dOut) || missing(g, dX) || !dW || !dw_s || !dw_t)
        RGNN_FAIL(RGNN_EINVAL, "a required tensor pointer is NULL");
    if (!workspace || !saved) RGNN_FAIL(RGNN_EWORKSPACE, "workspace or saved is NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int D = desc->d_out, K = desc->d_in;
    RgatBwdWs w; RgatSaved sv; RgatRunBwdWs rw;
    const bool runs = rgat_run_rows(g, desc);
    Bf16Stage stg(workspace, runs ? carve_rgat_run_bwd(g, desc, workspace, &rw) : carve_rgat_bwd(g, desc, workspace, &w), desc->dtype == RGNN_BF16, st);
    X = stg.in(X, (size_t)g->N * K);
    W = stg.in(W, (size_t)g->R * K * D);
    w_s = stg.in(w_s, (size_t)g->R * D);
    w_t = stg.in(w_t, (size_t)g->R * D);
    dOut = stg.in(dOut, (size_t)g->N * D);
    RGNN_TRY(stg.status);
    if (runs)
        return rgat_run_bwd(g, desc, static_cast<const float*>(X), static_cast<const float*>(W), static_cast<const float*>(w_s), static_cast<const float*>(w_t),
                            saved, static_cast<const float*>(dOut), static_cast<float*>(dX), dW, dw_s, dw_t, rw, st);
    carve_rgat_saved(g, desc, const_cast<void*>(saved), &sv);
    const float* Xf = static_cast<const float*>(X);
    const float* Wf = static_cast<const float*>(W);
    if (rgat_keeps_runs(g, desc)) {              // (a flag asked for rows per pair)
        TypedLinearArgs a{};
        a.tiles = pair_chunks(g, D).f32; a.X = Xf; a.gather = g->idx[RGNN_IDX_PAIR_SRC]; a.W = Wf; a.Y = sv.Hs = w.Hs; a.sign_matters = 1;
        RGNN_TRY(typed_linear_fwd(K, D, a, st));
    }
    const float* dO = static_cast<const float*>(dOut);
    const bool acc = grads_accumulate(desc);
    GradAcc ga;
    dW = ga.route(w.acc_dW, dW, (size_t)g->R * K * D);
    dw_s = ga.route(w.acc_dws, dw_s, (size_t)g->R * D);
    dw_t = ga.route(w.acc_dwt, dw_t, (size_t)g->R * D);
    const float* dX_old = acc ? static_cast<const float*>(dX) : nullptr;      // added by the kernel that writes dX
    // U[h][r]: the relations whose runs were walked in pieces (step 3), added with the shares of the weight gradients
    ShareSums sums;
    sums.pieces = SumArgs{w.run_partial, g->relrun_items.split_row, g->relrun_items.split_ptr, w.U, (size_t)g->relrun_items.num_partials * K,
                           (size_t)g->R * K, g->relrun_items.num_split, K, desc->heads};
    if (desc->heads > 1) {
        const int H = desc->heads;
        const float *ws = static_cast<const float*>(w_s), *wt = static_cast<const float*>(w_t);
        // 1. per CSR edge and head: att recomputed from the gathered row and the saved (m, s), and
        //    dz = att (dOut[v].Hs[pair_e] - dOut[v].out[v])_h * (z > 0 ? 1 : slope);  adz[e] = (att[0..H), dz[0..H))
        //    With the row selector the only edge of a single-edge pair also writes that pair's (dz[0..H), att[0..H)) into
        //    ds_src[p], which holds 2 H floats per pair.
        const bool sel = rgat_row_select(desc);
        RGNN_TRY(rgat_edge_dot_bwd(g, D, H, sv.Hs, ws, sv.s_dst, sv.ms, dO, static_cast<const float*>(out), desc->slope, w.adz,
                                   nullptr, nullptr, sel ? w.ds_src : nullptr, st));
        // 2. per-head sums of dz over runs and over pairs: ds_src[p][h] is element p * 2 H + h (step 1 wrote the pairs
        //    with one edge when the selector is on)
        //    (in the same launch the vectors W[r] w_t[r] per head for step 7)
        const FoldArgs fold = fold_args(g->R, K, D, H, Wf, wt, w.wtp);
        RGNN_TRY(segment_scalar_sum((int)g->Q, g->idx[RGNN_IDX_RUN_PTR], g->long_runs, nullptr, w.adz, 2 * H, H, w.ds_dst, st,
                                    "ds_dst_sum", 0, H, false, 0, &fold));
        RGNN_TRY(segment_scalar_sum((int)g->P, g->idx[RGNN_IDX_OUT_PTR], g->long_pairs, g->idx[RGNN_IDX_OUT_EPOS], w.adz, 2 * H, H,
                                    w.ds_src, st, "ds_src_sum", sel ? 2 : 0, H, sel, 2 * H));
        // 3. dHs[p] = sum_{e in out(p)} att_e dOut[dst_e] (per head)  +  ds_src[p][h] w_s[r] (per head).  With the
        //    selector only for the pairs with several edges (step 4 forms the other rows from dOut as it reads them),
        //    and the walk sums ds_src[p][h] itself over the same (att, dz) entries; step 2 then covered only the pairs
        //    with more edges than a lane sums, among them the ones the walk cuts into pieces.
        //    The same launch then forms U[h][r] = sum over r's runs of ds_dst[q][h] X[run_dst[q]] for step 6.
        const Rank1 r1{w.ds_src, 2 * H, g->idx[RGNN_IDX_PAIR_REL], ws};      // the second term, added when a pair's row is stored
        if (sel)
            RGNN_TRY(rgat_bwd_walks(g, RgatBwdWalks{K, D, H, w.adz, dO, w.G, w.ds_src, 2 * H, ws, w.partial, w.ds_dst, Xf, w.U, w.run_partial}, st));
        else
            RGNN_TRY(gather_sum(g->pair_items, D, g->idx[RGNN_IDX_OUT_EPOS], g->idx[RGNN_IDX_OUT_DST], 0, w.adz, 2 * H, 0, dO, w.G, w.partial,
                                st, 1, "aggregate_bwd_pair", "aggregate_bwd_pair.combine", H, 0, 0, &r1));
        // 4. dXp = dHs W^T, dW = sum X^T dHs; with the selector also A[r][h] = sum over r's pairs of ds_src[p][h] X[src_p]
        TypedLinearBwdArgs b{};
        b.tiles = pair_chunks(g, D).f32_bwd; b.X = Xf; b.gather = g->idx[RGNN_IDX_PAIR_SRC]; b.W = Wf; b.dY = w.G; b.dXrow = w.dXp;
        b.dW = static_cast<float*>(dW); b.part = w.tl_part;
        if (sel) { b.ysel = g->pair_ysel; b.dY_alt = dO; b.hcoef = w.ds_src; b.wvec = ws; b.sel_heads = H; b.Avec = w.A; b.sums = &sums; }
        RGNN_TRY(typed_linear_bwd(K, D, b, st));
        if (sel) RGNN_TRY(sums.launch(st));
        // 5. dw_s[r] = sum over r's pairs of ds_src[p][h] Hs[p] (per head; the pair rows are in relation order);
        //    with the selector from A instead, in step 6: dw_s[r] = (A[r][h] W[r]) on the columns of head h
        // 6. U as above;  dw_t and the w_t part of dW from it
        if (!sel) {
            RGNN_TRY(gather_sum(g->relpair_items, D, nullptr, nullptr, 0, w.ds_src, 2 * H, 0, sv.Hs, dw_s, w.partial, st, 2,
                                "src_vec_grad", "src_vec_grad.combine", H));
            RGNN_TRY(gather_heads_rows(g->relrun_items, K, H, g->R, g->idx[RGNN_IDX_RELRUN_IDX], g->relrun_dst, 0, w.ds_dst,
                                       Xf, w.U, w.run_partial, st, "dst_side_wgrad", "dst_side_wgrad.combine"));
        }
        const RgatFinish fin{g->R, K, D, H, Wf, ws, wt, sel ? w.A : nullptr, w.U, static_cast<float*>(dW), static_cast<float*>(dw_s),
                             static_cast<float*>(dw_t), 0};
        // 7. dX[u] = sum over u's pairs of dXp + sum over u's runs and heads of ds_dst[q][h] (W[r] w_t[r])_h
        RGNN_TRY(node_grad_sum(g, K, w.dXp, w.ds_dst, w.wtp, dX_old, dX, st, 0, 0, H, nullptr, &fin));
        return ga.flush(st);
    }
    // 1. per CSR edge: (att_e, dz_e), att_e recomputed from the gathered row and the saved (m, s); for single-edge pairs also ds_src[p] and G[p] = att_e dOut[dst_e] (or, with
    //    the row selector, only att_e: step 4 then reads the row from dOut).  With the selector ds_src[p] and that
    //    att_e are stored side by side (one 8-byte store here, one 8-byte load per row in step 4): w.ds_src then
    //    holds P pairs of floats and ds_src[p] is element 2 p.
    const bool sel = rgat_row_select(desc);
    const int dss = sel ? 2 : 1;
    RGNN_TRY(rgat_edge_dot_bwd(g, D, 1, sv.Hs, static_cast<const float*>(w_s), sv.s_dst, sv.ms, dO, static_cast<const float*>(out),
                               desc->slope, w.adz, w.G, w.ds_src, sel ? w.ds_src : nullptr, st));
    // 2. ds_dst[q] = sum over the run's edges of dz; in the same launch the folded vectors W[r] w_s[r] (step 4) and W[r] w_t[r] (step 6)
    const FoldArgs fold = fold_args(g->R, K, D, 1, Wf, static_cast<const float*>(w_s), w.wsp, static_cast<const float*>(w_t), w.wtp);
    RGNN_TRY(segment_scalar_sum((int)g->Q, g->idx[RGNN_IDX_RUN_PTR], g->long_runs, nullptr, w.adz, 2, 1, w.ds_dst, st, "ds_dst_sum", 0, 1,
                                false, 0, &fold));
    // 3. for the pairs with several edges (step 1 wrote the others): G[p] = sum_{e in out(p)} att_e dOut[dst_e] and, in
    //    the same walk over (att_e, dz_e), ds_src[p] = sum of dz_e; the pairs with more edges than a lane sums
    //    (among them the ones the walk cuts into pieces) get ds_src from the workgroup-per-segment sum afterwards
    //    Also U[r] = sum over r's runs of ds_dst[q] X[run_dst[q]] (step 4 adds the pieces of the relations that are cut)
    RGNN_TRY(rgat_bwd_walks(g, RgatBwdWalks{K, D, 1, w.adz, dO, w.G, w.ds_src, dss, nullptr, w.partial, w.ds_dst, Xf, w.U, w.run_partial}, st));
    RGNN_TRY(segment_scalar_sum((int)g->P, g->idx[RGNN_IDX_OUT_PTR], g->long_pairs, g->idx[RGNN_IDX_OUT_EPOS], w.adz, 2, 1, w.ds_src, st,
                                "ds_src_sum", 2, 1, true, dss));
    // 4. with dHs[p] = G[p] + ds_src[p] w_s[r]:
    //    dXp[p] = dHs[p] W[r]^T = G[p] W[r]^T + ds_src[p] (W[r] w_s[r]);  dW[r] = sum X^T G (+ A^T (x) w_s in step 5);
    //    A[r] = sum ds_src X
    TypedLinearBwdArgs b{};
    b.tiles = pair_chunks(g, D).f32_bwd; b.X = Xf; b.gather = g->idx[RGNN_IDX_PAIR_SRC]; b.W = Wf; b.dY = w.G; b.dXrow = w.dXp;
    b.rowscale = sel ? nullptr : w.ds_src; b.vec = w.wsp; b.dW = static_cast<float*>(dW); b.Avec = w.A;
    b.part = w.tl_part; b.sums = &sums;
    if (sel) { b.ysel = g->pair_ysel; b.dY_alt = dO; b.ds_yscale = reinterpret_cast<const float2*>(w.ds_src); }
    RGNN_TRY(typed_linear_bwd(K, D, b, st));
    RGNN_TRY(sums.launch(st));
    // 5. dw_s = A W, dw_t = U W, dW += A^T (x) w_s + U^T (x) w_t
    const RgatFinish fin{g->R, K, D, 1, Wf, static_cast<const float*>(w_s), static_cast<const float*>(w_t), w.A, w.U, static_cast<float*>(dW),
                         static_cast<float*>(dw_s), static_cast<float*>(dw_t), 0};
    // 6. dX[u] = sum over u's pairs of dXp + sum over u's runs of ds_dst[q] (W[r] w_t[r])
    RGNN_TRY(node_grad_sum(g, K, w.dXp, w.ds_dst, w.wtp, dX_old, static_cast<float*>(dX), st, 0, 0, 1, nullptr, &fin));
    return ga.flush(st);
}

// =========================================================================== HGT

extern "C" rgnn_status_t rgnn_hgt_fwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* desc, const void* X,
                                      const void* Wk, const void* Wq, const void* Wv, const void* Wo, const void* Watt,
                                      const void* Wmsg, const void* mu, void* out, void* saved, void* workspace,
                                      void* stream) {
    RGNN_TRY(check_desc(g, desc, RGNN_LAYER_HGT));
    ScheduleFlagsScope sched_scope(desc->flags);
    if (missing(g, X) || !Wk || !Wq || !Wv || !Wo || !Watt || !Wmsg || missing(g, out)) RGNN_FAIL(RGNN_EINVAL, "a required tensor pointer is NULL");
    if (!workspace) RGNN_FAIL(RGNN_EWORKSPACE, "workspace is NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int D = desc->d_out, H = desc->heads;
    HgtFwdWs w; HgtSaved sv;
    const bool bf16 = desc->dtype == RGNN_BF16, h = rows_bf16(desc);
    const void *X16 = bf16 ? X : nullptr, *Wk16 = bf16 ? Wk : nullptr, *Wq16 = bf16 ? Wq : nullptr,
               *Wv16 = bf16 ? Wv : nullptr, *Wo16 = bf16 ? Wo : nullptr;
    const size_t carved = carve_hgt_fwd(g, desc, workspace, &w);
    saved = saved_or_scratch(g, RGNN_LAYER_HGT, desc, saved, workspace, carved);
    Bf16Stage stg(workspace, carved, bf16, st);
    const size_t tdd = (size_t)g->T * D * D;
    // fp32 copies of what the fp32 kernels read (below width 128; the kernels on weights alone read the caller's storage)
    const bool fold = hgt_folded(g, desc);
    const float* X32 = !h ? stg.in(X, (size_t)g->N * D) : nullptr;
    const float* Wk32 = !h && !fold ? stg.in(Wk, tdd) : nullptr;
    const float* Wq32 = !h ? stg.in(Wq, tdd) : nullptr;
    const float* Wv32 = !h && !fold ? stg.in(Wv, tdd) : nullptr;
    const float* Wo32 = !h ? stg.in(Wo, tdd) : nullptr;
    RGNN_TRY(stg.status);
    const HgtWeights hw{Wk, Wv, Watt, Wmsg, mu, bf16, g->rel_src_type, D, H};
    carve_hgt_saved(g, desc, saved, &sv);
    const int32_t* perm = g->idx[RGNN_IDX_NTYPE_PERM];
    const int32_t* psrc = g->idx[RGNN_IDX_PAIR_SRC];
    // bf16 form of an intermediate row tensor (nullptr when the rows are fp32) and its fp32 form
    auto R16 = [h](const void* p) { return h ? p : nullptr; };
    auto R32 = [h](const void* p) { return h ? nullptr : static_cast<const float*>(p); };
    // Row products of one step, which do not depend on each other: one launch where they are built as one (fp32 rows up to width
    // 64), a launch each otherwise.
    struct Product { bool pairs; const void* in; const void* w32; const void* w16; void* out; const char* label; };
    void* const Mrow = h ? static_cast<void*>(static_cast<uint16_t*>(sv.KM) + D) : static_cast<void*>(static_cast<float*>(sv.KM) + D);
    auto products = [&](std::initializer_list<Product> list, const char* label) -> rgnn_status_t {
        if (bf16 || D == 128) {
            for (const Product& p : list)
                RGNN_TRY(tl_fwd(bf16, p.pairs ? pair_chunks(g, D) : node_chunks(g, D), D, p.in == X ? X32 : R32(p.in), p.in == X ? X16 : R16(p.in),
                                p.pairs ? psrc : perm, !p.pairs, static_cast<const float*>(p.w32), p.w16, p.out, h, p.label, st, 0, p.pairs ? 2 : 1));
            return RGNN_OK;
        }
        TypedLinearArgs a[3] = {};
        int n = 0;
        for (const Product& p : list) {
            TypedLinearArgs& t = a[n++];
            t.tiles = jobs_fwd_list(p.pairs ? pair_chunks(g, D) : node_chunks(g, D));
            t.X = static_cast<const float*>(p.in); t.gather = p.pairs ? psrc : perm; t.scatter_out = !p.pairs;
            t.W = static_cast<const float*>(p.w32); t.Y = static_cast<float*>(p.out); t.y_stride = p.pairs ? 2 : 1;
        }
        return typed_linear_fwd_jobs(D, a, n, label, st);
    };
    // 1. per node type: Q, and K, V unless they are folded into the per-pair linears
    // 2. compact per pair, side by side in KM[p]: Ka[p] = K[src_p] Watt[r], M[p] = V[src_p] Wmsg[r]
    const Product q{false, X, Wq32, Wq16, sv.Q, "node_linear_q"};
    if (fold) {
        //    = X[src_p] (Wk[type of r's sources] Watt[r]) and X[src_p] (Wv[type] Wmsg[r])
        //    With bf16 rows the products are rounded to bf16 once (as K and V would have been) and feed the
        //    matrix cores as they are; rows in the storage of the intermediates: the caller's bf16 X at width
        //    128, its fp32 copy otherwise.
        RGNN_TRY(hgt_fold(g->R, hw, sv.Wf_att, sv.Wf_msg, h, st));
        const void* in = h ? X : static_cast<const void*>(X32);
        if (h) {
            RGNN_TRY(products({q}, ""));
            RGNN_TRY(typed_linear_fwd_bf16({&g->pair_tiles_cu1, X, psrc, 0, sv.Wf_att, sv.Wf_msg, sv.KM, "pair_linear"}, st));
        } else RGNN_TRY(products({q, {true, in, R32(sv.Wf_att), R16(sv.Wf_att), sv.KM, "pair_linear_att"},
                           {true, in, R32(sv.Wf_msg), R16(sv.Wf_msg), Mrow, "pair_linear_msg"}}, "node_pair_linears"));
    } else {
        //    with the per-(relation, head) matrices as block-diagonal d x d weights
        RGNN_TRY(hgt_expand(g->R, hw, w.Wbd_att, w.Wbd_msg, st));
        RGNN_TRY(products({q, {false, X, Wk32, Wk16, sv.K, "node_linear_k"}, {false, X, Wv32, Wv16, sv.V, "node_linear_v"}}, "node_linears"));
        RGNN_TRY(products({{true, sv.K, w.Wbd_att, nullptr, sv.KM, "pair_linear_att"}, {true, sv.V, w.Wbd_msg, nullptr, Mrow, "pair_linear_msg"}},
                          "pair_linears"));
    }
    // 3. one walk per destination: logit per edge and head, softmax over the destination's edges, Z[v][h] = sum_e att[e][h] M[pair_e][h]
    RGNN_TRY(hgt_attend_fwd(g, D, H, sv.KM, sv.Q, sv.Z, sv.ms, w.partial, w.part_ms, st, h));
    // 4. out = Z Wo[type]
    RGNN_TRY(tl_fwd(bf16, node_chunks(g, D), D, R32(sv.Z), R16(sv.Z), perm, 1, Wo32, Wo16, out, false, "node_linear_out", st));
    return RGNN_OK;
}

extern "C" rgnn_status_t rgnn_hgt_bwd(const rgnn_graph_t* g, const rgnn_layer_desc_t* desc, const void* X,
                                      const void* Wk, const void* Wq, const void* Wv, const void* Wo, const void* Watt,
                                      const void* Wmsg, const void* mu, const void* out, const void* saved,
                                      const void* dOut, void* dX, void* dWk, void* dWq, void* dWv, void* dWo,
                                      void* dWatt, void* dWmsg, void* dmu, void* workspace, void* stream) {
    (void)out;
    RGNN_TRY(check_desc(g, desc, RGNN_LAYER_HGT));
    ScheduleFlagsScope sched_scope(desc->flags);
    if (missing(g, X) || !Wk || !Wq || !Wv || !Wo || !Watt || !Wmsg || missing(g, dOut) || missing(g, dX) || !dWk || !dWq || !dWv || !dWo || !dWatt || !dWmsg)
        RGNN_FAIL(RGNN_EINVAL, "a required tensor pointer is NULL");
    if (mu && !dmu) RGNN_FAIL(RGNN_EINVAL, "dmu is NULL but mu is given");
    if (!workspace || !saved) RGNN_FAIL(RGNN_EWORKSPACE, "workspace or saved is NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int D = desc->d_out, H = desc->heads;
    HgtBwdWs w; HgtSaved sv;
    const bool bf16 = desc->dtype == RGNN_BF16, h = rows_bf16(desc);
    const void *Wk16 = bf16 ? Wk : nullptr, *Wq16 = bf16 ? Wq : nullptr, *Wv16 = bf16 ? Wv : nullptr,
               *Wo16 = bf16 ? Wo : nullptr;
    Bf16Stage stg(workspace, carve_hgt_bwd(g, desc, workspace, &w), bf16, st);
    const size_t tdd = (size_t)g->T * D * D, rh = (size_t)g->R * H, dh = D / H;
    const bool fold = hgt_folded(g, desc);
    const float* X32 = !h ? stg.in(X, (size_t)g->N * D) : nullptr;
    const float* Wk32 = !h && !fold ? stg.in(Wk, tdd) : nullptr;
    const float* Wq32 = !h ? stg.in(Wq, tdd) : nullptr;
    const float* Wv32 = !h && !fold ? stg.in(Wv, tdd) : nullptr;
    const float* Wo32 = !h ? stg.in(Wo, tdd) : nullptr;
    const HgtWeights hw{Wk, Wv, Watt, Wmsg, mu, bf16, g->rel_src_type, D, H};
    const float* dO32 = !h ? stg.in(dOut, (size_t)g->N * D) : nullptr;
    RGNN_TRY(stg.status);
    carve_hgt_saved(g, desc, const_cast<void*>(saved), &sv);
    // row operands in the storage of this mode: the caller's bf16 tensors as they are, or the fp32 copies
    const void* Xr = h ? X : static_cast<const void*>(X32);
    const void* dOr = h ? dOut : static_cast<const void*>(dO32);
    const int32_t* perm = g->idx[RGNN_IDX_NTYPE_PERM];
    const int32_t* psrc = g->idx[RGNN_IDX_PAIR_SRC];
    const bool acc = grads_accumulate(desc);
    GradAcc ga;
    dWk = ga.route(w.acc_node[0], dWk, tdd); dWq = ga.route(w.acc_node[1], dWq, tdd);
    dWv = ga.route(w.acc_node[2], dWv, tdd); dWo = ga.route(w.acc_node[3], dWo, tdd);
    dWatt = ga.route(w.acc_rel[0], dWatt, rh * dh * dh); dWmsg = ga.route(w.acc_rel[1], dWmsg, rh * dh * dh);
    dmu = ga.route(w.acc_mu, dmu, rh);
    // 1. output linear: dZ = dOut Wo^T, dWo = Z^T dOut (the shares of the weight gradients are added by one launch, before their
    //    first use)
    ShareSums sums;
    RGNN_TRY(tl_bwd(h, node_chunks(g, D), D, sv.Z, perm, 1, Wo32, Wo16, dOr, w.dZ, h, static_cast<float*>(dWo), w.node_part[0],
                    "node_linear_out_bwd", st, false, nullptr, nullptr, nullptr, 0, 1, &sums));
    // 2. per destination: att (recomputed) and d logit per edge and head, dQ[v][h] = sum dl Ka[pair][h]
    RGNN_TRY(hgt_attend_bwd(g, D, H, sv.KM, sv.Q, sv.Z, sv.ms, w.dZ, w.dQ, w.adl, w.partial, st, h));
    // 3. per pair: dKa[p][h] = sum dl Q[dst][h], dM[p][h] = sum att dZ[dst][h]
    RGNN_TRY(hgt_pair_bwd(g, D, H, sv.Q, w.dZ, w.adl, w.dKM, w.partial, st, h));
    const void* dKa = w.dKM;
    const void* dM = h ? static_cast<const void*>(static_cast<const uint16_t*>(w.dKM) + D) : static_cast<const void*>(static_cast<const float*>(w.dKM) + D);
    // 4. per-pair linears backward
    if (fold) {
        // the folded weights take the per-pair gradients straight to X's rows; their own gradients are
        // unfolded into those of the node-type and of the per-relation matrices
        if (h) {
            //   dKp[p] = dKa Wf_att^T + dM Wf_msg^T in one kernel, with both weight gradients
            TypedLinearBwdBf16Args b{};
            b.tiles = &g->pair_tiles_cu1; b.X = X; b.gather = psrc; b.W = sv.Wf_att; b.W2 = sv.Wf_msg; b.w_bf16 = 1; b.dY = w.dKM;
            b.dy_stride = 2; b.dXrow = w.dKp; b.dW = w.dWf_att; b.dW2 = w.dWf_msg; b.part = w.pair_part[0]; b.label = "pair_linear_bwd"; b.sums = &sums;
            RGNN_TRY(typed_linear_bwd_bf16(D, b, st));
            if (hgt_pairs_with_query(g, desc)) {
                // dX = dQ Wq^T + sums over each node's pairs, with dWq
                TypedLinearBwdBf16Args q{};
                q.tiles = &g->node_tiles_sum; q.X = X; q.gather = perm; q.both_gathered = 1; q.W = Wq16; q.w_bf16 = 1; q.dY = w.dQ;
                q.dXrow = dX; q.dx_f32 = 1; q.accumulate = acc; q.dW = static_cast<float*>(dWq); q.part = w.node_part[1]; q.label = "node_linear_q_bwd";
                q.sum_ptr = g->idx[RGNN_IDX_SRCPAIR_PTR]; q.sum_row = g->idx[RGNN_IDX_SRCPAIR_IDX]; q.sum_rows = w.dKp; q.sums = &sums;
                RGNN_TRY(typed_linear_bwd_bf16(D, q, st));
            }
        } else if (!hgt_bwd_jobs(g, desc)) {
            RGNN_TRY(tl_bwd(false, pair_chunks(g, D), D, Xr, psrc, 0, static_cast<const float*>(sv.Wf_att), nullptr, dKa, w.dKp, false, w.dWf_att,
                            w.pair_part[0], "pair_linear_att_bwd", st, false, nullptr, nullptr, nullptr, 0, 2, &sums));
            RGNN_TRY(tl_bwd(false, pair_chunks(g, D), D, Xr, psrc, 0, static_cast<const float*>(sv.Wf_msg), nullptr, dM, w.dVp, false, w.dWf_msg,
                            w.pair_part[1], "pair_linear_msg_bwd", st, false, nullptr, nullptr, nullptr, 0, 2, &sums));
        }
        // dX = dQ Wq^T + sums over each node's pairs of the two per-pair gradients
        if (hgt_bwd_jobs(g, desc)) {
            TypedLinearBwdArgs b[3] = {};
            for (int k = 0; k < 2; ++k) {
                b[k].tiles = hgt_pair_list(g, D); b[k].gather = psrc; b[k].W = static_cast<const float*>(k ? sv.Wf_msg : sv.Wf_att);
                b[k].dY = static_cast<const float*>(k ? dM : dKa); b[k].dy_stride = 2; b[k].dXrow = static_cast<float*>(k ? w.dVp : w.dKp);
                b[k].dW = k ? w.dWf_msg : w.dWf_att; b[k].part = w.pair_part[k];
            }
            b[2].tiles = hgt_node_list(g, D); b[2].gather = perm; b[2].dy_gathered = b[2].scatter_dx = 1; b[2].W = Wq32;
            b[2].dY = static_cast<const float*>(w.dQ); b[2].dXrow = w.dXq; b[2].dW = static_cast<float*>(dWq); b[2].part = w.node_part[1];
            for (TypedLinearBwdArgs& x : b) { x.X = static_cast<const float*>(Xr); x.sums = &sums; }
            RGNN_TRY(typed_linear_bwd_jobs(D, b, 3, "node_pair_linears_bwd", st));
        } else if (!hgt_pairs_with_query(g, desc)) {
            RGNN_TRY(tl_bwd(h, node_chunks(g, D), D, Xr, perm, 1, Wq32, Wq16, w.dQ, w.dXq, false, static_cast<float*>(dWq),
                            w.node_part[1], "node_linear_q_bwd", st, false, nullptr, nullptr, nullptr, 0, 1, &sums));
        }
        RGNN_TRY(sums.launch(st));
        RGNN_TRY(hgt_fold_bwd(g->T, g->R, hw, w.dWf_att, w.dWf_msg, static_cast<float*>(dWk), static_cast<float*>(dWv),
                              static_cast<float*>(dWatt), static_cast<float*>(dWmsg), static_cast<float*>(dmu), st));
        if (hgt_pairs_with_query(g, desc)) return ga.flush(st);
        if (acc) RGNN_TRY(add_into((size_t)g->N * D, static_cast<const float*>(dX), w.dXq, st));
        RGNN_TRY(node_grad_sum(g, D, w.dKp, nullptr, nullptr, w.dXq, dX, st, h, 0, 1, h ? nullptr : w.dVp));
        return ga.flush(st);
    }
    RGNN_TRY(hgt_expand(g->R, hw, w.Wbd_att, w.Wbd_msg, st));
    RGNN_TRY(tl_bwd(h, pair_chunks(g, D), D, sv.K, psrc, 0, w.Wbd_att, nullptr, dKa, w.dKp, h, w.dWbd_att, w.pair_part[0],
                    "pair_linear_att_bwd", st, false, nullptr, nullptr, nullptr, 0, 2, &sums));
    RGNN_TRY(tl_bwd(h, pair_chunks(g, D), D, sv.V, psrc, 0, w.Wbd_msg, nullptr, dM, w.dVp, h, w.dWbd_msg, w.pair_part[1],
                    "pair_linear_msg_bwd", st, false, nullptr, nullptr, nullptr, 0, 2, &sums));
    RGNN_TRY(sums.launch(st));
    RGNN_TRY(hgt_extract(g->R, hw, w.dWbd_att, w.dWbd_msg, static_cast<float*>(dWatt), static_cast<float*>(dWmsg),
                         static_cast<float*>(dmu), st));
    // 5. dK[u], dV[u] = sums over u's pairs
    RGNN_TRY(node_grad_sum(g, D, w.dKp, nullptr, nullptr, nullptr, w.dK, st, h, h));
    RGNN_TRY(node_grad_sum(g, D, w.dVp, nullptr, nullptr, nullptr, w.dV, st, h, h));
    // 6. node linears backward and dX
    //    (bf16 rows: the three input gradients are accumulated into dX by the kernels themselves)
    RGNN_TRY(tl_bwd(h, node_chunks(g, D), D, Xr, perm, 1, Wk32, Wk16, w.dK, h ? dX : static_cast<void*>(w.dXk),
                    false, static_cast<float*>(dWk), w.node_part[0], "node_linear_k_bwd", st, h && acc, nullptr, nullptr, nullptr, 0, 1, &sums));
    RGNN_TRY(tl_bwd(h, node_chunks(g, D), D, Xr, perm, 1, Wq32, Wq16, w.dQ, h ? dX : static_cast<void*>(w.dXq),
                    false, static_cast<float*>(dWq), w.node_part[1], "node_linear_q_bwd", st, h, nullptr, nullptr, nullptr, 0, 1, &sums));
    RGNN_TRY(tl_bwd(h, node_chunks(g, D), D, Xr, perm, 1, Wv32, Wv16, w.dV, h ? dX : static_cast<void*>(w.dXv),
                    false, static_cast<float*>(dWv), w.node_part[2], "node_linear_v_bwd", st, h, nullptr, nullptr, nullptr, 0, 1, &sums));
    RGNN_TRY(sums.launch(st));
    if (!h) {
        if (acc) RGNN_TRY(add_into((size_t)g->N * D, static_cast<const float*>(dX), w.dXk, st));
        RGNN_TRY(add3((size_t)g->N * D, w.dXk, w.dXq, w.dXv, static_cast<float*>(dX), st));
    }
    return ga.flush(st);
}
