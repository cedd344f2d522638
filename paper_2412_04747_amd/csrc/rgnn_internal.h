// Internal declarations shared by the library's translation units (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <algorithm>
#include <string>
#include <vector>
#include "../../include/rgnn.h"
#include "work_lists.h"

namespace rgnn {

// ---- error plumbing ------------------------------------------------------
void set_error(const char* fmt, ...);
#define RGNN_HIP(call)                                                                  \
    do {                                                                                \
        hipError_t e_ = (call);                                                         \
        if (e_ != hipSuccess) {                                                         \
            rgnn::set_error("%s failed: %s (%s:%d)", #call, hipGetErrorString(e_), __FILE__, __LINE__); \
            return RGNN_EHIP;                                                           \
        }                                                                               \
    } while (0)
#define RGNN_FAIL(code, ...)          \
    do {                              \
        rgnn::set_error(__VA_ARGS__); \
        return (code);                \
    } while (0)
#define RGNN_TRY(expr)                      \
    do {                                    \
        rgnn_status_t s_ = (expr);          \
        if (s_ != RGNN_OK) return s_;       \
    } while (0)

// ---- optional kernel timing (profile.hip) ----------------------------------
class KernelTimer {
  public:
    KernelTimer(hipStream_t st, const char* name);
    ~KernelTimer();
  private:
    hipStream_t st_;
    int idx_;
};

// ---- work lists ----------------------------------------------------------
// Runs that one of the eight half wavefronts of a destination takes one after the other (rgcn_small.hip), and their edges.
struct RunChain {
    int32_t runs = 0, edges = 0;
    int64_t length() const { return edges + 32 * (int64_t)runs; }      // in edges: a run costs about as much as 32 of them
};
// Row tiles of a segmented row range (rows grouped by relation or node type),
// cut into `num_chunks` contiguous chunks, one per persistent workgroup.  A
// chunk owns one partial-gradient slot per distinct segment it touches; slots
// are numbered in (chunk, segment) order, which is also segment order, so the
// slots of one segment are contiguous (seg_slot_ptr).
struct TileList {
    int32_t tile_rows = 0;       // rows per tile
    int32_t num_tiles = 0;
    int32_t num_chunks = 0;
    int32_t num_slots = 0;
    int32_t num_segs = 0;
    int32_t max_seg_slots = 0;       // slots of the segment with the most
    int32_t max_chunk_slots = 0;     // ... and of the chunk
    // chunks of as many tiles but very different numbers of segments, each with its weight load (and flush): the chunks of the long
    // relations are done early
    bool uneven() const { return 2 * (int64_t)max_chunk_slots * num_chunks > 3 * (int64_t)num_slots; }
    int32_t* tile_seg = nullptr;     // [num_tiles]  device
    int32_t* tile_row0 = nullptr;    // [num_tiles]  first row of the tile
    int32_t* tile_row1 = nullptr;    // [num_tiles]  end row (exclusive; <= row0 + tile_rows)
    int32_t* chunk_tile = nullptr;   // [num_chunks+1]
    int32_t* chunk_slot = nullptr;   // [num_chunks]  first slot of the chunk
    int32_t* seg_slot_ptr = nullptr; // [num_segs+1]
};

// Segments of a CSR-like list cut into items of at most `max_len` entries.  An
// item is either a whole segment (slot < 0: the result goes to row `row`) or a
// piece of a split segment (slot >= 0: the result goes to partial row `slot`;
// split_* lists say which partial rows sum to which output row).
struct ItemList {
    int32_t num_items = 0;
    int32_t num_partials = 0;
    int32_t num_split = 0;
    int32_t* beg = nullptr;        // [num_items]
    int32_t* end = nullptr;        // [num_items]
    int32_t* row = nullptr;        // [num_items] segment id
    int32_t* slot = nullptr;       // [num_items] partial row or -1
    int32_t* split_row = nullptr;  // [num_split]
    int32_t* split_ptr = nullptr;  // [num_split+1] range of partial rows
    int32_t* part_item = nullptr;  // [num_partials] item that writes the partial row
    int32_t num_long = 0;
    int32_t* long_item = nullptr;  // [num_long] items with more than kSerialMax entries, and every piece of a cut segment
    int32_t* part_split = nullptr; // [num_partials] index into split_* of its segment
    int32_t first_single = 0;      // items [first_single, first_single + num_single) are the whole segments
    int32_t num_single = 0;        // with exactly one entry
    int32_t first_short = 0;       // items [first_short, first_short + num_short) are the whole segments with
    int32_t num_short = 0;         // 2..kShortLen entries; the single-entry ones follow directly
    int32_t num_wide = 0;          // items [0, num_wide) have kWideMin entries or more
};

}  // namespace rgnn

namespace rgnn {
// Ids of the segments of a CSR-like list that are longer than kSerialMax entries.
struct LongList {
    int32_t n = 0;
    int32_t* ids = nullptr;
};
}  // namespace rgnn

struct rgnn_graph {
    int64_t N = 0, E = 0, P = 0, Q = 0;
    int32_t R = 0, T = 0;
    int num_cus = 0;                       // compute units of the device the graph lives on
    int64_t max_in_degree = 0, max_pair_out_degree = 0, num_single_pairs = 0;
    rgnn::RunChain longest_chain;          // (an upper bound above 131072 runs)
    size_t index_bytes = 0;
    int32_t* idx[RGNN_IDX_COUNT] = {};     // device arrays, see RGNN_IDX_*
    int64_t idx_len[RGNN_IDX_COUNT] = {};
    float* in_invc = nullptr;              // [E] 1 / c_{v,r} per CSR edge
    float* out_invc = nullptr;             // [E] the same per pair-major edge: in_invc[out_epos[j]]
    rgnn::TileList pair_tiles;             // pairs segmented by relation
    rgnn::TileList node_tiles;             // nodes (in ntype_perm order) segmented by type
    rgnn::TileList all_tiles;              // all nodes as one segment (RGCN self-loop)
    rgnn::TileList pair_tiles_wide;        // same tiles as pair_tiles / node_tiles in fewer, longer chunks: for the
    rgnn::TileList node_tiles_wide;        // forward kernels whose chunks each load, or split, an fp32 weight
    rgnn::TileList pair_tiles_cu2;         // the same in one chunk per workgroup of a kernel that keeps two (one)
    rgnn::TileList pair_tiles_cu1;         // workgroups per compute unit
    rgnn::TileList node_tiles_cu2;
    rgnn::TileList node_tiles_cu1;
    rgnn::TileList all_tiles_cu1;
    rgnn::TileList pair_tiles_hgt;         // the shares of two lists of the pairs and one of the nodes in one chunk per compute unit
    rgnn::TileList node_tiles_hgt;         // for all three together
    rgnn::TileList pair_tiles_loop;        // likewise one list of the pairs and one of all nodes (RGCN with a self-loop)
    rgnn::TileList all_tiles_loop;
    rgnn::ItemList dst_items;              // CSR edges by destination
    rgnn::ItemList pair_items;             // transposed edges by pair
    rgnn::ItemList pair_items_multi;       // the same, pairs with two or more edges only
    rgnn::ItemList srcpair_items;          // pairs by source node (never cut)
    int32_t max_node_pairs = 0;            // most pairs of a source node
    rgnn::TileList node_tiles_sum;         // node tiles by type, in chunks of like numbers of rows and pairs (HGT: the pairs' sum with the query's product)
    int32_t* in_pair_tag = nullptr;        // [E] in_pair with the top bit set when the pair has a single edge
    float* pair_scale = nullptr;           // [P] 1 / c_{v,r} of the only edge of a single-edge pair, 1 for the other pairs
    int32_t* pair_ysel = nullptr;          // [P] pair id, or for a pair with one edge the top bit | that edge's destination
    int32_t* relrun_dst = nullptr;         // [Q] destination of the runs in (relation, destination) order: run_dst[relrun_idx[i]]
    int32_t* rel_src_type = nullptr;       // [R] node type of the sources of relation r (0 for a relation without edges)
    bool rel_src_tied = false;             // every relation's sources are of one node type (rel_src_type is then valid)
    rgnn::ItemList relrun_items;           // runs by relation
    rgnn::ItemList relpair_items;          // pairs by relation (rows of the compact tensors are already in this order)
    // Rows per (destination, relation) run instead of per (source, relation) pair (run_rows; schedule.h).  The rows are in (relation,
    // several edges before one, destination) order.
    bool run_rows = false;
    int64_t num_multi_runs = 0, num_single_runs = 0;
    int64_t rows_saved = 0;                // by rows per run over a training step (schedule.h)
    int32_t* run_tag = nullptr;            // [Q] the run, with the top bit set when it has several edges
    int32_t* multi_run = nullptr;          // [num_multi_runs] run of each number
    int32_t* row_in = nullptr;             // [Q] by row: source of the run's only edge, or the top bit | number of the run among those
                                           // with several edges, in run order
    int32_t* row_dst = nullptr;            // [Q] by row: destination
    int32_t* src_row = nullptr;            // [E] by (source, relation, CSR position): row of the edge's run
    float* src_invc = nullptr;             // [E] 1 / c_{v,r} of that edge
    int32_t *src_run = nullptr, *src_rel = nullptr;       // [E] its run, with the top bit set when it is the run's only edge, and its relation
    int32_t* in_spos = nullptr;            // [E] place in that order of a CSR edge
    int32_t* pair_spos = nullptr;          // [P] and of a pair's first edge
    int32_t* row_run = nullptr;            // [Q] run of a row
    rgnn::TileList run_tiles_wide, run_tiles_cu1, run_tiles_loop, all_tiles_run_loop;   // as those of the pairs
    rgnn::ItemList multi_run_items;        // CSR edges of the runs with several edges (row: their number)
    rgnn::ItemList dstrun_items;           // runs by destination
    rgnn::ItemList src_items;              // edges by source
    rgnn::ItemList pair_blocks, run_blocks;               // pairs, and runs, by relation and block of nodes (plan_blocks)
    rgnn::LongList long_runs;              // runs (run_ptr) too long for one lane
    rgnn::LongList long_pairs;             // pairs (out_ptr) too long for one lane
    std::vector<void*> allocs;             // every device allocation, for destroy
};

namespace rgnn {

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// Raises a kernel's dynamic LDS limit once per (kernel, device) instead of on every launch.
rgnn_status_t allow_dynamic_lds(const void* kernel, size_t bytes);

// Device address of the library's static scratch buffer on the current device (layers.hip); resolved once per device.
rgnn_status_t static_scratch(void** p);

// weight folds (fold_weight_block in device_utils.h), as a launch or `blocks` workgroups of another one
struct FoldArgs { const float* W; const float* w; const float* w2; int R, kd, nd, H; float* wv; float* wv2; int blocks; };

// ---- kernel launchers (typed_linear.hip) --------------------------------
struct TypedLinearArgs {
    const TileList* tiles;
    const float* X;          // input rows
    const int32_t* gather;   // row i reads X[gather[i]] (nullptr: X[i])
    const float* W;          // [segs][KD][ND]
    float* Y;                // output rows
    int scatter_out;         // 1: row i writes Y[gather[i]], 0: Y[i]
    int accumulate;          // 1: Y += result
    const float* vec;        // optional [segs][ND]: s_out[i][h] = Y_row . vec[seg] over the h-th of s_heads column slices
    float* s_out;            // [rows][s_heads]
    int s_heads = 1;         // a power of two with ND / s_heads >= 16
    const char* label;       // name in the timing report (nullptr: default)
    int y_stride = 1;        // rows of Y are y_stride * d_out floats apart (1 or 2)
    int relu = 0;            // with accumulate: Y = max(Y + result, 0)
    const FoldArgs* fold = nullptr;   // folds weights in the same launch (gathered rows, no scatter, accumulate or vec)
    const float* X2 = nullptr;        // gather[i] < 0: row i reads X2[gather[i] & 0x7FFFFFFF] (plain products of gathered rows); row i of the
    const int32_t* to = nullptr;      // result is then row to[i] of Y
    int sign_matters = 0;    // 1: a backward takes a branch on the sign of what becomes of Y (leaky ReLU; ReLU, also the caller's own)
};
rgnn_status_t typed_linear_fwd(int d_in, int d_out, const TypedLinearArgs& a, hipStream_t st);

// pieces of D floats (a multiple of 16), `copies` sets of them, summed per cut segment
struct SumArgs {
    const float* partial; const int32_t* split_row; const int32_t* split_ptr; float* out;
    size_t partial_copy, out_copy;       // floats from one set to the next
    int num_split, D, copies;
    __host__ __device__ int64_t blocks() const { return (int64_t)num_split * copies * (D / 16); }
};
// What backward typed linears leave to be summed: dW[s] (kn floats) and, when given, dW2[s] (kd floats) = sums of segment s's slots of
// kn + kd floats each, for up to kMax lists, and optionally two sets of pieces as above.  One launch (traversal.hip) sums them all.
struct ShareSums {
    static constexpr int kMax = 4;
    enum { kMany, kUneven, kFew };           // how a list's slots lie (traversal.hip)
    struct Job {
        const float* part; const int32_t* seg_slot_ptr;
        int blocks, col_blocks, kind, kn, kd, used;      // used: floats of a slot that are summed
        float* dW; float* dW2;
    };
    Job job[kMax];
    int n = 0;
    SumArgs pieces{}, pieces2{};
    rgnn_status_t add(const TileList& tiles, const float* part, int kn, int kd, float* dW, float* dW2);
    rgnn_status_t launch(hipStream_t st);      // and is empty again
};
struct TypedLinearBwdArgs {
    const TileList* tiles;
    const float* X;          // forward input rows
    const int32_t* gather;   // forward gather (nullptr: identity)
    const float* W;          // [segs][KD][ND]
    const float* dY;         // gradient of the forward output
    int dy_gathered;         // 1: row i reads dY[gather[i]], 0: dY[i]
    float* dXrow;            // [rows][KD] per-row input gradient dY_i W^T (row i, or gather[i] if scatter_dx)
    int scatter_dx;
    const float* rowscale;   // optional [rows]: A[seg] = sum_i rowscale[i] X_row_i
    const float* vec;        // optional [segs][KD] (with rowscale): dXrow[i] += rowscale[i] * vec[seg]
    float* dW;               // [segs][KD][ND]
    float* Avec;             // [segs][KD] (with rowscale); [segs][sel_heads][KD] = sum over the rows of hcoef[i][h] X[g(i)] (with hcoef)
    float* part;             // scratch [num_slots][KD*ND + KD]
    const char* label;
    // Optional row selector (widths up to 64, ungathered dY): row i of dY is
    // ysel[i] < 0 ? scale_i * dY_alt[ysel[i] & 0x7FFFFFFF] : dY[ysel[i]].  With `vec`, rowscale[i] and scale_i come
    // interleaved as ds_yscale[i] = (rowscale_i, scale_i) and `rowscale` stays null; without, scale_i is yscale[i], or 1
    // where yscale is null (either way scale_i counts only where the top bit of ysel[i] is set).
    const int32_t* ysel = nullptr;
    const float* dY_alt = nullptr;
    const float2* ds_yscale = nullptr;
    const float* yscale = nullptr;
    // Per-head row selector (widths up to 64, sel_heads in {2, 4}, instead of rowscale / vec / ds_yscale): a selected
    // row is dY_alt[row] * a[h] + b[h] * wvec[seg] on the columns of head h, (b[0..H), a[0..H)) = hcoef[i] for row i
    const float* hcoef = nullptr;    // [rows][2][sel_heads]
    const float* wvec = nullptr;     // [segs][ND]
    int sel_heads = 0;
    const float* X2 = nullptr;       // gather[i] < 0: row i of X is X2[gather[i] & 0x7FFFFFFF]; row i of dY is dY[ysel[i]] (no dY_alt); with
                                     // yscale the X row counts yscale[num[i]] times in dW, and rowdot[num[i]] = dXrow[i] . yscale[num[i]] X row
    float* rowdot = nullptr;
    const int32_t* num = nullptr;
    int dy_stride = 1;               // rows of dY are dy_stride * d_out floats apart (1 or 2)
    ShareSums* sums = nullptr;       // the slots are left to the caller's sums (part then has to last until they are launched)
};
// bf16 matrix-core variant (typed_linear_bf16.hip): Y[i] = A[g(i)] W[seg]
struct TypedLinearBf16Args {
    const TileList* tiles;
    const void* A;           // rows: bf16 (a_bf16) or fp32
    int a_bf16;
    const int32_t* gather;   // row i reads A[gather[i]] (nullptr: A[i])
    int scatter_out;         // 1: row i writes Y[gather[i]]
    const void* W;           // [segs][d][d]: bf16 (w_bf16) or fp32
    int w_bf16;
    void* Y;                 // output rows: bf16 (y_bf16) or fp32
    int y_bf16;
    const char* label;
    int y_stride = 1;        // rows of Y are that many widths apart
};
rgnn_status_t typed_linear_bf16(int d, const TypedLinearBf16Args& a, hipStream_t st);
// width 128, all rows and weights in bf16 (typed_linear_fwd_bf16.hip): Y[i] = X[gather[i]] W[seg], or with a second weight
// (X[gather[i]] W[seg], X[gather[i]] W2[seg]) in rows 256 wide
struct TypedLinearFwdBf16Args {
    const TileList* tiles; const void* X; const int32_t* gather; int scatter_out; const void* W; const void* W2; void* Y; const char* label;
};
rgnn_status_t typed_linear_fwd_bf16(const TypedLinearFwdBf16Args& a, hipStream_t st);

// Backward on the bf16 matrix cores (typed_linear_bwd_bf16.hip): X, dY and (unless dx_f32) dXrow rows in bf16.
struct TypedLinearBwdBf16Args {
    const TileList* tiles;
    const void* X;
    const int32_t* gather;   // row i reads X[gather[i]]
    int both_gathered;       // 1: dY rows are read and dXrow rows written through the gather list as well
    const void* W;           // [segs][d][d]: bf16 (w_bf16) or fp32
    int w_bf16;
    const void* W2 = nullptr;   // optional second weight (bf16) for the second half of dY rows two widths wide
    const void* dY;
    int dy_stride = 1;       // rows of dY are that many widths apart
    void* dXrow;             // dY W^T (+ dY2 W2^T)
    int dx_f32 = 0;
    int accumulate = 0;      // fp32 dXrow += result
    float* dW;               // [segs][d][d]
    float* dW2 = nullptr;
    float* part;             // scratch: num_slots * d * d floats per weight
    const char* label;
    // optional row selector for dY (ungathered dY only): row i is dY[ysel[i]], or dY_alt[ysel[i] & 0x7FFFFFFF]
    // when the top bit of ysel[i] is set; with yscale it is also multiplied by yscale[i]
    const int32_t* ysel = nullptr;
    const void* dY_alt = nullptr;
    const float* yscale = nullptr;
    // optional (bf16 weight, fp32 dXrow gathered on both sides): dXrow[n] += the rows sum_row[sum_ptr[n] .. sum_ptr[n + 1]) of sum_rows
    const int32_t* sum_ptr = nullptr;
    const int32_t* sum_row = nullptr;
    const void* sum_rows = nullptr;
    ShareSums* sums = nullptr;   // as in TypedLinearBwdArgs
};
rgnn_status_t typed_linear_bwd_bf16(int d, const TypedLinearBwdBf16Args& a, hipStream_t st);
// the slots of a list go to the caller's sums, or are summed by a launch of their own (sums null)
rgnn_status_t typed_linear_slot_reduce(const TileList& tiles, const float* part, int kn, int kd, float* dW, float* dW2, hipStream_t st,
                                       ShareSums* sums);

size_t typed_linear_bwd_scratch_floats(int d_in, int d_out, const TileList& t, int vectors = 1);   // vectors: of a slot's vector part
rgnn_status_t typed_linear_bwd(int d_in, int d_out, const TypedLinearBwdArgs& a, hipStream_t st);
// RGCN, widths 32 and 64: the pairs' backward and the self-loop's (ungathered rows) in one launch, both with sums
rgnn_status_t typed_linear_bwd_loop(int d_in, int d_out, const TypedLinearBwdArgs& pair, const TypedLinearBwdArgs& loop, hipStream_t st);
// up to three products of gathered rows in one launch, widths 32 and 64: rows scattered back the same way, or two widths apart
rgnn_status_t typed_linear_fwd_jobs(int d, const TypedLinearArgs* a, int n, const char* label, hipStream_t st);
rgnn_status_t typed_linear_bwd_jobs(int d, const TypedLinearBwdArgs* a, int n, const char* label, hipStream_t st);   // with sums
// width 128 (typed_linear_split.hip): fp32 operands split into three bf16 planes; the backward fills the slots only
rgnn_status_t typed_linear_split_fwd(const TypedLinearArgs& a, hipStream_t st);
rgnn_status_t typed_linear_split_bwd(const TypedLinearBwdArgs& a, hipStream_t st);

}  // namespace rgnn
