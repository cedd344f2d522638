// Per-graph, per-layer choice of schedule and layout: which of the alternative kernels and data
// layouts a layer call uses, decided from the statistics of the graph index and the layer
// descriptor (the thesis' point that no single schedule / layout fits every graph, Ch.3 "Compact
// Tensor Materialization and Data Layout" and the evaluation's per-dataset comparison of the
// optimizations).  Plain C++, no device code: layers.hip and the traversal launchers call these
// predicates where they pick a kernel, rgnn_schedule reports them, and the host tests exercise
// this header on its own.
#pragma once
#include <stddef.h>
#include <stdint.h>
#include "../../include/rgnn.h"

namespace rgnn {

// A list of segments gets a batched walk of its single-entry (2..4-entry) whole segments only when it holds
// this many of them: below that the extra kernel phase costs more than the general walk loses on them.
constexpr int kBatchedMin = 4096;
// w_s of single-head RGAT (R x d fp32) stays in LDS for the fused traversal up to this size; beyond it the
// walks read it through the caches.
constexpr size_t kWsLdsMax = 64 * 1024;

inline bool flag_set(uint32_t flags, uint32_t bit) { return (flags & bit) != 0; }

// number of whole segments of one kind the batched walk takes (0: they stay with the general walk)
inline int batched_count(int count, uint32_t flags) {
    return (!flag_set(flags, RGNN_FLAG_NO_BATCHED_WALKS) && count >= kBatchedMin) ? count : 0;
}
// bf16 inputs at width 128: every row tensor (inputs, intermediates, saved tensors, incoming gradients) is bf16 storage
inline bool sched_rows_bf16(int dtype, int d) { return dtype == RGNN_BF16 && d == 128; }
// The gradient row of a (source, relation) pair with one edge is not materialised: the typed-linear backward reads
// it from the destination's gradient row through a row selector.  Built for RGAT with one head, and up to width 64 with two
// or four (the fused fp32 backward kernel); and for RGCN, with bf16 rows and, with fp32 rows, where the walk it saves is longer
// than what it adds to the backward: a run of a relation's rows then starts with one load more, selector before row.  Backward
// with / without, us: width 64, 50 relations 38 / 38 at 30k edges (16k such pairs), 194 / 237 at 1M; 500 of equal frequency 43 / 41 at
// 10k, 75 / 76 at 100k (198 such pairs per relation), 141 / 155 at 400k; 2000 129 / 123 at 100k (50), 159 / 157 at 200k (99), 194 /
// 208 at 400k (198); 4000 243 / 243 at 200k (50), 281 / 313 at 400k (99: the rows of the pairs no longer fit the caches); width 32, 4000 139
// / 135 at 400k, 176 / 201 at 1M; width 128, where the loads run two units ahead, 500 51 / 50 at 10k, 61 / 63 at 30k, 2000 252 / 278 at 200k.
// Where most edges lie in other pairs: 4 relations, 200k edges, 10 % in such pairs 46.6 / 43.8 (width 64), 1M edges 126.7 / 127.4.
inline bool sched_row_select(int layer, int dtype, int d, int heads, int R, int64_t edges, int64_t single_pairs, uint32_t flags) {
    if (flag_set(flags, RGNN_FLAG_NO_ROW_SELECT)) return false;
    if (layer == RGNN_LAYER_RGAT) return heads == 1 || (d <= 64 && (heads == 2 || heads == 4) && d % (4 * heads) == 0);
    if (layer == RGNN_LAYER_RGCN)
        return sched_rows_bf16(dtype, d) ||
               (single_pairs * d >= 640000 && (d == 128 || ((single_pairs >= 160 * (int64_t)R || single_pairs * d >= 24000000) &&
                                                            (6 * single_pairs >= edges || single_pairs * d >= 4000000))));
    return false;
}
// Rows per (destination, relation) run instead of per (source, relation) pair.  Where destinations are popular and sources are not, a graph
// has fewer runs than pairs; summing a run's inputs before the product, and multiplying a run's gradient row once, then moves fewer
// rows: 2 E + 7 Q - 2 Q1 over a training step (Q runs, Q1 of them with one edge, which are read where they are) against
// 2 E + 7 P - 2 P1, and has fewer products.  The graph gets the lists for it where that is so (sched_run_rows).
// RGCN, forward + backward, us, pairs / runs, at 7 Q - 2 Q1 from 0.54 to 0.72 of 7 P - 2 P1: 300k edges, 60 relations, width 32 81 / 81, 64
// 145 / 126, 128 277 / 211; 3M edges 443 / 340, 930 / 649, 2283 / 1438; at equal numbers 78 / 76, 140 /
// 139 and 273 / 268 (300k edges); at 1.7 times the rows 172 / 205 (width 128, 8 relations).  Below 131072 edges the sum, a
// launch or two more, costs what the rest saves: 100k edges 56 / 56, 85 / 88, 131 / 126.
// Not where rows are stored in bf16 (layers.hip): a row of a run is a partial sum of out, and the sum of a run's inputs a partial sum of dW;
// both were rounded to bf16 once, which rows per pair do not do (error of out with 64 edges per run and non-negative features 1.7e-3 for 3.4e-4).
inline bool sched_run_rows(int64_t edges, int64_t pairs, int64_t single_pairs, int64_t runs, int64_t single_runs) {
    return edges >= (1 << 17) && 20 * (7 * runs - 2 * single_runs) <= 19 * (7 * pairs - 2 * single_pairs);
}
// Rows per run walk the edges over rows of the input width, rows per pair over those of the output width, so with narrower outputs the rows
// saved (of the formula above) have to make up for the edges' longer ones.  64 -> 32, forward + backward, pairs / runs by rows saved per edge:
// RGCN 0.81 to 0.87 of the time at 0.03 to 0.2 from 1.25M edges on, 0.93 to 0.95 at 0.37 to 0.43, 0.98 to 1.03 at 0.48 to 0.74, 1.0 to 1.3
// above; RGAT 0.89 to 1.01 up to 0.42, 0.96 to 1.04 at 0.5 to 0.75, 1.0 to 1.18 above.  (32 -> 64: 1.05 to 1.6 throughout.)
inline bool sched_run_widths(int d_in, int d_out, int64_t edges, int64_t rows_saved) { return d_in <= d_out || 20 * rows_saved >= 9 * edges; }
// The calls that take them.  Every flag but the accumulation of gradients asks for an alternative of the rows per pair.
inline bool sched_use_run_rows(bool lists, uint32_t flags) { return lists && !(flags & ~(uint32_t)RGNN_FLAG_ACCUMULATE); }
inline bool sched_rgcn_run_rows(bool lists, int64_t edges, int d, uint32_t flags) { return sched_use_run_rows(lists, flags) && edges * d >= 8000000; }
// RGCN forwards that keep nothing for a backward: the saving has to come from the forward alone.  Pairs / runs, us: 300k edges, 60
// relations, width 32 34 / 46, 64 59 / 64, 128 129 / 109; 1M 75 / 73, 145 / 124, 340 / 266.
inline bool sched_run_rows_infer(int64_t edges, int d) { return edges * d >= 30000000; }
// Workgroups that finish the parameter gradients of RGAT (traversal.hip), and how many go with run_term's (512 threads each).
inline int64_t finish_blocks(int R, int d_in, int d) { return (int64_t)R * (d / 32 + (d_in * d + 1023) / 1024); }
constexpr int64_t kMaxFinishBlocks = 1 << 22;
// RGAT with one head.  The walks look the relations' folded vectors up, once per run or edge, so more relations move the line out, and at
// width 32 the indices outweigh the rows.  Forward + backward, us, pairs / runs, at 7 Q - 2 Q1 from 0.54 to 0.72 of 7 P - 2 P1: 8 relations,
// width 64 173 / 152 at 300k edges, 1108 / 798 at 3M, 128 178 / 162 at 140k, 463 / 338 at 550k; 60 relations, 64 300 / 260 at 550k, 1317 / 990 at 3M, 128
// 213 / 217 at 140k, 352 / 306 at 300k, 2873 / 1930 at 3M, 32 175 / 182 at 550k, 307 / 292 at 1.2M; 400 relations, 64 396 / 440 at 550k, 683 / 683
// at 1.2M, 1533 / 1380 at 3M, 128 451 / 485 at 300k, 1394 / 1220 at 1.2M, 32 788 / 838 at 3M.
// Not with so many relations that the workgroups which finish their gradients in run_term's launch would leave few of the 2^32 lanes of a grid.
inline bool sched_rgat_run_rows(bool lists, int heads, int R, int64_t edges, int d, uint32_t flags) {
    return heads == 1 && sched_use_run_rows(lists, flags) && edges * d >= 16000000 + (int64_t)R * (d < 64 ? 640000 : 160000) &&
           finish_blocks(R, d, d) <= kMaxFinishBlocks;
}
// ... and for forwards that keep nothing for a backward, where the softmax within the runs is paid and the cheaper backward is not there.  Pairs / runs
// as a ratio: width 64 1.04 and 1.02 (8 and 60 relations, 1.2M and 3M edges), 0.99 and 0.90 at 550k, 400 relations 0.90 at 3M; 128 1.11 and 1.08 at
// 550k, 0.99 and 1.00 at 300k, 400 relations 1.00 at 1.2M and 1.06 at 3M; 32 0.93 at 3M.
inline bool sched_rgat_run_rows_infer(int R, int64_t edges, int d) { return d >= 64 && edges * d >= 64000000 + (int64_t)R * 640000; }
// HGT: the key and message linears of the nodes are folded into the per-relation weights when every relation's
// sources have one node type.
inline bool sched_hgt_folded(bool rel_src_tied, uint32_t flags) {
    return rel_src_tied && !flag_set(flags, RGNN_FLAG_NO_WEIGHT_FOLDING);
}
// HGT, rows in bf16: the sum over a node's pairs in the query's product (typed_linear_bwd_bf16.hip, PAIRS) where nodes have few, and none
// has many (32 rows wait for the one with most).  The walk's gathers are wider; what is saved is a row of fp32 per node, written and read.
// Layer, forward + backward, us, walk / in the product: at 1.2 pairs per node 380 / 367 (120k nodes), 1241 / 1169 (500k); 1.5 167 / 165 (30k); 2.7
// 318 / 320 (60k), 515 / 515 (120k), 10375 / 10100 (2M); 4.5 414 / 416 (60k), 719 / 722 (120k); 5 3004 / 2955 (500k), 5967 / 5929 (1M); 6.3
// 2398 / 2394 (300k); 15 4345 / 4416 (300k); 31 2558 / 2627 (60k).
inline bool sched_hgt_pairs_with_query(int64_t nodes, int64_t pairs, int most) {
    return pairs > 0 && most <= 32 && (pairs <= 2 * nodes || (pairs <= 5 * nodes && nodes >= 150000));
}
// RGAT: edge softmax fused into the aggregation walk (otherwise, one head only, a pass of its own that stores one
// attention weight per edge); the edge-parallel comparison schedule needs the per-edge weights
inline bool sched_fused_softmax(uint32_t flags) {
    return !flag_set(flags, RGNN_FLAG_SEPARATE_SOFTMAX) && !flag_set(flags, RGNN_FLAG_EDGE_PARALLEL_AGGREGATION);
}
// RGAT, rows per pair: the destination halves of the logits with the folded vectors of all relations and heads in LDS, one workgroup of 1024
// threads per compute unit or more, where the runs are many for what each of them then loads.  From memory / from LDS, us, width 64, four
// heads: 100 relations 7.3 / 8.0 at 59k runs, 14.0 / 12.0 at 207k, 55 / 33 at 1.1M; 30 relations 7.2 / 6.3 at 51k; width 128 45 / 29 at 429k.
inline bool sched_halves_in_lds(int R, int heads, int d, int64_t runs) {
    return (size_t)R * heads * d * sizeof(float) <= 150 * 1024 && runs >= 1024 * (int64_t)R;
}
inline bool sched_ws_in_lds(int R, int d) { return (size_t)R * d * sizeof(float) <= kWsLdsMax; }

// RGCN forward of a small graph in one launch (rgcn_small.hip), which reads a weight per (relation, destination) run, and one per
// node for the self-loop, where the general plan reads one per tile of rows; a workgroup per destination, whose eight half wavefronts
// take its runs in turn, each run walked by one of them.  Two lines, both in the cost of a run (its product and its rows: linear in the
// weight's and the row's length), and both further out where the general plan has more launches: destinations that it cuts into
// pieces (17 us for 10 at 10k edges), a self-loop.
//   throughput  runs and nodes (a workgroup's start and end cost as much as two runs).  One launch / general plan, us: no self-loop, nothing
//               cut, 32 x 32 7.9 / 12.9 at 1000 nodes and 5.7k runs, 9.7 / 11.4 at 4000 and 18k, 11.5 / 10.8 at 8192 and 15k; 64 x 64 9.6 / 14.2 at
//               2000 and 6.9k, 15.3 / 12.6 at 4000 and 10k; with cut destinations 32 x 32 15.4 / 19.4 at 4000 and 24k, 16.6 / 18.8 at 20k and 10k, 64
//               x 64 22 / 22 at 6700 and 12k; with both 32 x 32 18.4 / 23.1 at 13k and 17k, 64 x 64 24.6 / 27.1 at 4000 and 10k, 27.6 / 25.4 at 10k
//               and 5.7k.
//   latency     the longest chain of a half wavefront (long ones belong to cut destinations).  Eight destinations of n edges, n relations: 32
//               x 32 11.7 / 15.3 at 64 (chains of 8), 20 / 15 at 128; 64 x 64 11.6 / 15.1 at 32, 21 / 18 at 64.  Runs and edges of the chain:
//               64 x 64 13.2 / 19 at 1 and 188, 18.1 / 19.9 at 5 and 117, 19.6 / 20.3 at 8 and 32; 32 x 32 18.7 / 16.8 at 15 and 23; with a
//               self-loop 64 x 64 20.2 / 25.3 at 1 and 300, 22.8 / 23.5 at 9 and 16, 34 / 24.5 at 12 and 15.
// Over 720 graphs of 1k to 40k edges, four pairs of widths, with and without a self-loop, the pick takes 0.6 % longer than the faster of the
// two on average (always one launch 15 %, never 73 %).
inline bool sched_rgcn_small(int dtype, int d_in, int d, bool self_loop, int64_t runs, int64_t nodes, bool cut, int64_t chain_runs,
                             int64_t chain_edges, uint32_t flags) {
    if (dtype != RGNN_F32 || d_in > 64 || d > 64 || flag_set(flags, RGNN_FLAG_NO_BATCHED_WALKS)) return false;
    const int64_t kd = d_in * d, run = kd + 48 * d_in + 1024;
    const int64_t most = (self_loop ? 128000000 + 12000 * kd : 90000000 + 8000 * kd) * (cut ? 13 : 10) / 10;
    const int64_t longest = self_loop ? 40800 + 680 * d_in : 33600 + 560 * d_in;
    return (2 * runs + (self_loop ? 5 : 4) * nodes) * run <= 2 * most && chain_runs * run + chain_edges * (7 * d_in / 2) <= longest;
}

struct ListCounts { int32_t single = 0, short_ = 0; };   // whole segments with 1 / with 2..kShortLen entries
struct ScheduleIn {
    int layer = 0, dtype = 0, d = 0, heads = 1;
    uint32_t flags = 0;
    int R = 1;
    int64_t edges = 0;
    bool rel_src_tied = false;
    int item_len = 0, tile_chunks = 0, wide_chunks = 0;
    ListCounts dst, pair, pair_multi;     // destination-major list, pair-major list, pair-major list of multi-edge pairs
};

inline rgnn_schedule_t pick_schedule(const ScheduleIn& in) {
    rgnn_schedule_t s{};
    s.item_len = in.item_len;
    s.tile_chunks = in.tile_chunks;
    s.wide_chunks = in.wide_chunks;
    s.rows_bf16 = sched_rows_bf16(in.dtype, in.d) && in.layer != RGNN_LAYER_RGAT;
    s.row_select = sched_row_select(in.layer, in.dtype, in.d, in.heads, in.R, in.edges, in.pair.single, in.flags);
    s.hgt_folded = in.layer == RGNN_LAYER_HGT && sched_hgt_folded(in.rel_src_tied, in.flags);
    s.fused_softmax = in.layer == RGNN_LAYER_RGAT && sched_fused_softmax(in.flags);
    s.ws_in_lds = s.fused_softmax && sched_ws_in_lds(in.R, in.d);
    s.edge_parallel = in.layer == RGNN_LAYER_RGAT && flag_set(in.flags, RGNN_FLAG_EDGE_PARALLEL_AGGREGATION);
    s.dst_batched_single = batched_count(in.dst.single, in.flags) > 0;
    s.dst_batched_short = batched_count(in.dst.short_, in.flags) > 0;
    // the pair-major backward walk runs over the multi-edge pairs only where the row selector (or, for single-head
    // RGAT, the edge walk itself) serves the single-edge pairs
    const bool multi_only = s.row_select || (in.layer == RGNN_LAYER_RGAT && in.heads == 1);
    const ListCounts& pl = multi_only ? in.pair_multi : in.pair;
    s.pair_batched_single = batched_count(pl.single, in.flags) > 0;
    s.pair_batched_short = batched_count(pl.short_, in.flags) > 0;
    s.pair_walk_multi_only = multi_only;
    return s;
}

}  // namespace rgnn
