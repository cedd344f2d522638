// Launchers of the traversal kernels (traversal.hip).  Internal.
#pragma once
#include "rgnn_internal.h"

namespace rgnn {

// desc.flags of the layer call in progress on this thread: the launchers consult it where they choose between
// the batched and the general walk (set by the entry points for the duration of a call).
uint32_t current_schedule_flags();
struct ScheduleFlagsScope {
    explicit ScheduleFlagsScope(uint32_t flags);
    ~ScheduleFlagsScope();
    uint32_t prev;
};

// wv[r] = W[r] w[r]; optionally a second vector per relation in the same pass (wv2[r] = W[r] w2[r]).  H > 1: wv[r][h], over the
// columns of head h
FoldArgs fold_args(int R, int kd, int nd, int H, const float* W, const float* w, float* wv, const float* w2 = nullptr, float* wv2 = nullptr);
rgnn_status_t fold_weight(const FoldArgs& f, hipStream_t st);
// Folds go into another kernel's launch while their workgroups leave most of the 2^32 lanes of a grid to that kernel, whose workgroups
// may have 512 threads (it saves a launch of some microseconds; with as many folds as this one the launch takes milliseconds).
inline bool fold_rides(const FoldArgs& f) { return f.blocks <= 1 << 22; }
rgnn_status_t segment_scalar_sum(int n, const int32_t* ptr, const LongList& lng, const int32_t* via, const float* val,
                                 int stride, int off, float* out, hipStream_t st, const char* label, int min_len = 0,
                                 int heads = 1, bool long_only = false, int ostride = 0,     // ostride 0: heads
                                 const FoldArgs* with_fold = nullptr);                      // folds weights in the same launch
// ms (optional, [N] pairs of floats): (max, sum of exp) of the logits of every destination with edges
rgnn_status_t edge_softmax(const rgnn_graph* g, const float* s_src, const float* s_dst, float slope, float* att,
                           float* part_m, float* part_s, hipStream_t st, float* ms = nullptr);
// rgat_fused.hip: RGAT (H heads; head h owns column slice h) with the edge softmax fused into the traversal.
//   forward: out[v] = sum_e att_e Hs[pair_e] per head, att = softmax over v's edges of leakyrelu(Hs[pair_e] . w_s[r_e] + s_dst[run_e][h]);
//   ms[v][h] = (max logit, sum of exp(logit - max)) as pairs of floats; partial / part_ms: scratch rows and (m, s) pairs of the
//   pieces of cut destinations
rgnn_status_t rgat_aggregate_fwd(const rgnn_graph* g, int D, int H, const float* Hs, const float* w_s, const float* s_dst,
                                 float slope, float* out, float* ms, float* partial, float* part_ms, hipStream_t st);
//   backward: adz[e] = (att_e[0..H), dz_e[0..H)) with att_e recomputed from the gathered row and ms; one head: the only edge
//   of a single-edge pair also writes dsy[p] = (dz_e, att_e), or without dsy: ds_src[p] = dz_e and G[p] = att_e dOut[v]
rgnn_status_t rgat_edge_dot_bwd(const rgnn_graph* g, int D, int H, const float* Hs, const float* w_s, const float* s_dst,
                                const float* ms, const float* dOut, const float* out, float slope, float* adz, float* G,
                                float* ds_src, float* dsy, hipStream_t st);
// Rows per run, one head:
//   lq[q] = (logit, 1) of the runs with one edge, where the walk over the runs does not write it
rgnn_status_t rgat_single_logits(const rgnn_graph* g, int K, const float* X, const float* wsp, const float* s_dst, float slope, float* lq, hipStream_t st);
//   the inputs of the m-th run with several edges, A[m] = sum of X[src_e] weighted by their softmax within the run, from the logits
//   X[src_e] . wsp[r] + s_dst[q]; lq[q] = (max logit, sum of exp(logit - max)).  partial / part_ms: pieces of runs that are cut
rgnn_status_t rgat_run_inputs(const rgnn_graph* g, int K, const float* X, const float* wsp, const float* s_dst, float slope, float* A, float* lq,
                              float* partial, float* part_ms, hipStream_t st);
//   out[v] = sum over v's runs of their rows Y, a run weighing sum exp(logit - max over v); a run with one edge has the logit
//   Y . w_s[r] + s_dst[q], which becomes its lq[q] (may be null without such runs to be kept); ms[v] = (max, sum of exp)
rgnn_status_t rgat_run_aggregate(const rgnn_graph* g, int D, const float* Y, const float* w_s, const float* s_dst, float slope, float* lq, float* out,
                                 float* ms, float* partial, float* part_ms, hipStream_t st);
//   the destination halves of the logits, s_dst[q] = X[dst_q] . wtp[r]
rgnn_status_t rgat_run_logit(const rgnn_graph* g, int K, const float* X, const float* wtp, float* s_dst, hipStream_t st);
//   backward (rgat_runs.hip): weight[q] = what A[q] (or the source's row) counts in out[dst_q];
//   stat[q] = (s_dst[q], max of v, 1 / sum of v, dOut[v] . out[v] = sum over v's runs of rowdot), of a run with one edge (logit, max, 1 / sum, dz),
//   and ds_dst of those
rgnn_status_t rgat_run_weights(const rgnn_graph* g, const float* ms, const float* lq, float* weight, hipStream_t st);
rgnn_status_t rgat_run_stat(const rgnn_graph* g, float slope, const float* rowdot, const float* weight, const float* ms, const float* lq, const float* s_dst,
                            float* stat, float* ds_dst, hipStream_t st);
//   per source u, over its edges in the order of src_items: dz[i], and dX[u] = sum att_e dH[row of e's run] + dz_e wsp[r_e] (+ dX[u], acc;
//   dX NULL: dz alone),
//   with dH = dOut W^T per run
rgnn_status_t rgat_source_walk(const rgnn_graph* g, int K, const float* X, const float* dH, const float* wsp, const float* stat, float slope, float* dz,
                               float* dX, bool acc, float* partial, hipStream_t st);
//   A[r] = sum over r's pairs of ds_src X[src], ds_src the sum of the pair's dz (ds_src: scratch [P] for the long ones); U[r] = sum over r's
//   runs of ds_dst X[dst]; what the partials hold is left to the caller's sums (pair_blocks, run_blocks)
rgnn_status_t rgat_block_sums(const rgnn_graph* g, int K, const float* X, const float* dz, float* ds_src, const float* ds_dst, float* A, float* a_partial,
                              float* U, float* u_partial, hipStream_t st);
// workgroups of `threads` threads with `lds` bytes of dynamic LDS that stay resident per compute unit (cached per kernel)
rgnn_status_t resident_blocks_per_cu(const void* kernel, int threads, size_t lds, int* out);
// Optional rank-1 term of a gather-sum: out[i] += coef[i * stride + head] * vec[seg[i]] (fp32 vec rows of the output width)
struct Rank1 { const float* coef; int stride; const int32_t* seg; const float* vec; };
rgnn_status_t gather_sum(const ItemList& L, int D, const int32_t* via, const int32_t* rowidx, int row_by_k,
                         const float* coef, int cstride, int cabs, const void* src, void* out, float* partial,
                         hipStream_t st, int role, const char* label, const char* combine_label, int heads = 1,
                         int src_bf16 = 0, int out_bf16 = 0, const Rank1* r1 = nullptr,
                         const float* extra = nullptr);     // role 3: added to the output rows (may be out)
// RGAT's backward (heads 1, 2 or 4), one launch: for the pairs with several edges G[p] = sum_e att_e dOut[dst_e] (+ ds_src[p] ws[r] per
// head, with ws) and ds_src[p] = sum_e dz_e per head (element p * ds_src_stride + h; not for the pairs that are cut: the caller sums
// those); by relation U[h][r] = sum_q ds_dst[q][h] X[dst_q], whose cut relations stay as pieces in run_partial
// (ShareSums adds them).
struct RgatBwdWalks {
    int d_in, d_out, heads;
    const float* adz; const float* dOut; float* G; float* ds_src; int ds_src_stride; const float* ws; float* pair_partial;
    const float* ds_dst; const float* X; float* U; float* run_partial;
};
rgnn_status_t rgat_bwd_walks(const rgnn_graph* g, const RgatBwdWalks& a, hipStream_t st);
// rows of the cut segments of a list from their pieces: plain sums (widths 32 .. 256), and sums whose pieces carry their
// own softmax statistics (max, sum) per head.  copies: that many independent sets of partial rows (one after the other)
// and of output rows (out_copy elements apart).  full_exp: expf instead of __expf (bf16 rows: always).  The partial rows carry the factor
// pow2_share(piece_len) (device_utils.h).
rgnn_status_t combine_partials(const ItemList& L, int D, const float* partial, void* out, int out_bf16, const char* label,
                               hipStream_t st, const Rank1* r1 = nullptr, int heads = 1, int copies = 1, size_t out_copy = 0,
                               const float* extra = nullptr);
rgnn_status_t combine_softmax(const ItemList& L, int D, int H, const float* partial, const float* part_ms, void* out,
                              int out_bf16, float* ms, bool full_exp, int piece_len, const char* label, hipStream_t st,
                              const int32_t* ms_row = nullptr);      // (max, sum) of segment v at ms_row[v] instead of v
// H weighted sums of the same gathered rows in one walk (coef [entries][H]); out [H][out_rows][D]
rgnn_status_t gather_heads_rows(const ItemList& L, int D, int H, int out_rows, const int32_t* via, const int32_t* rowidx,
                                int row_by_k, const float* coef, const float* src, float* out, float* partial,
                                hipStream_t st, const char* label, const char* combine_label);
// RGAT's parameter gradients from A, U and the typed linear's share of dW (A null: dw_s is not formed)
struct RgatFinish {
    int R, kd, nd, H;
    const float* W; const float* w_s; const float* w_t; const float* A; const float* U;
    float* dW; float* dw_s; float* dw_t;
    int blocks;          // set by the launcher
};
//   dX[v] += sum over v's runs of ds_dst[q] wtp[r], and the parameter gradients
rgnn_status_t rgat_run_term(const rgnn_graph* g, int D, const float* ds_dst, const float* wtp, float* dX, RgatFinish fin, hipStream_t st);
rgnn_status_t node_grad_sum(const rgnn_graph* g, int D, const void* dXp, const float* ds_dst, const float* wtp,
                            const float* extra, void* dX, hipStream_t st, int in_bf16 = 0, int out_bf16 = 0, int heads = 1,
                            const void* dXp2 = nullptr, const RgatFinish* finish = nullptr);
// rgcn_small.hip: the whole forward of a small graph in one launch (fp32, widths 32 and 64)
rgnn_status_t rgcn_small_fwd(const rgnn_graph* g, int K, int D, const float* X, const float* W, const float* W0, int norm, int relu, float* out,
                             hipStream_t st);
// hgt.hip: the layer's weights in the caller's storage (fp32 or bf16); rel_type = node type of each relation's sources
struct HgtWeights { const void* Wk; const void* Wv; const void* Watt; const void* Wmsg; const void* mu; bool bf16; const int32_t* rel_type; int d; int H; };
//   folded weights of both halves: Wf_att[r] = Wk[rel_type[r]] blockdiag(mu / sqrt(dh) Watt[r]), Wf_msg[r] = Wv[..] blockdiag(Wmsg[r])
rgnn_status_t hgt_fold(int R, const HgtWeights& w, void* Wf_att, void* Wf_msg, int out_bf16, hipStream_t st);
//   and the gradients of all the weights from those of the folded ones (dWk, dWv: sums over a type's relations in ascending order)
rgnn_status_t hgt_fold_bwd(int T, int R, const HgtWeights& w, float* dWf_att, float* dWf_msg, float* dWk, float* dWv, float* dWatt,
                           float* dWmsg, float* dmu, hipStream_t st);
//   block-diagonal expansion of both per-(relation, head) weights (the attention one scaled) and its backward
rgnn_status_t hgt_expand(int R, const HgtWeights& w, float* Wbd_att, float* Wbd_msg, hipStream_t st);
rgnn_status_t hgt_extract(int R, const HgtWeights& w, float* dWbd_att, float* dWbd_msg, float* dWatt, float* dWmsg, float* dmu,
                          hipStream_t st);
// hgt_walk.hip: the edge walks of HGT over the key / message rows KM[p][2][D] of the pairs (rows fp32 or bf16)
//   forward: Z[v] = sum_e att_e M[pair_e], att = softmax per head of Ka[pair_e] . Q[v]; ms[v][h] = (max, sum of exp)
rgnn_status_t hgt_attend_fwd(const rgnn_graph* g, int D, int H, const void* KM, const void* Q, void* Z, float* ms,
                             float* partial, float* part_ms, hipStream_t st, int rows_bf16);
//   backward, destination-major: adl[e][h] = (att, dl), dl = att (dZ . M - dZ . Z); dQ[v] = sum_e dl Ka[pair_e]
rgnn_status_t hgt_attend_bwd(const rgnn_graph* g, int D, int H, const void* KM, const void* Q, const void* Z, const float* ms,
                             const void* dZ, void* dQ, float* adl, float* partial, hipStream_t st, int rows_bf16);
//   backward, pair-major: dKM[p] = (sum dl Q[dst], sum att dZ[dst]); partial rows are 2 D wide
rgnn_status_t hgt_pair_bwd(const rgnn_graph* g, int D, int H, const void* Q, const void* dZ, const float* adl, void* dKM,
                           float* partial, hipStream_t st, int rows_bf16);
// rgat_heads.hip: s_dst[q][h] = X[dst_q] . wtp[r][h]
rgnn_status_t run_logit(const rgnn_graph* g, int D, int H, const float* X, const float* wtp, float* s_dst, hipStream_t st);
// out[v] = sum_e |att_e| Hs[pair_e] edge by edge with atomic adds (zeroes out first); fp32 rows
rgnn_status_t aggregate_edge_parallel(const rgnn_graph* g, int D, const float* att, const float* Hs, float* out,
                                      hipStream_t st);
rgnn_status_t add3(size_t n, const float* a, const float* b, const float* c, float* out, hipStream_t st);

rgnn_status_t widen_bf16(size_t n, const uint16_t* src, float* dst, hipStream_t st);
rgnn_status_t add_into(size_t n, const float* src, float* dst, hipStream_t st);     // dst += src
rgnn_status_t relu_inplace(size_t n, float* x, hipStream_t st);
rgnn_status_t relu_grad(size_t n, const float* ref, const void* gin, void* y, hipStream_t st, int bf16 = 0, float* y32 = nullptr);

}  // namespace rgnn
