// Weight kernels of the HGT layer: folding of the node linears into the per-(relation, head) matrices, their
// block-diagonal expansion where folding does not apply, and the backward of both.  (Caption of the thesis figure "HGT
// and RGAT layer": attention of HGT is an edgewise dot product between the relation-transformed key of the source and
// the query of the destination; the message depends only on (source node, edge type), so both are stored once per pair.
// The edge walks are in hgt_walk.hip.)
//
// The weights are read in the caller's storage (fp32 or bf16), and each kernel serves the key / attention half and the
// value / message half in one launch (blockIdx.y): on graphs of up to a few million edges these launches were a tenth to a
// quarter of the layer (22 launches, 173 us, of a forward + backward on 2M edges in bf16; now 3 launches, 40 us).
//
// The d_head x d_head matrices W[r][h] act as one block-diagonal d x d matrix per relation, so that the
// relation-segmented typed-linear kernel serves them unchanged; with bf16 or fp32 inputs that kernel is bound by HBM
// traffic at these widths, so the extra zero blocks cost no time.
#include "rgnn_internal.h"
#include "traversal.h"
#include "device_utils.h"

namespace rgnn {

namespace {

__device__ __forceinline__ float weight(const float* p, size_t i) { return p[i]; }
__device__ __forceinline__ float weight(const bf16_t* p, size_t i) { return __uint_as_float((uint32_t)p[i] << 16); }

// One half of the layer's weights: x = 0 key / attention (scaled by mu / sqrt(dh)), x = 1 value / message.
template <typename T>
struct Halves {
    const T* node[2];        // [types][d][d]
    const T* rel[2];         // [R][H][dh][dh]
    const T* mu;             // [R][H] or null
    const int32_t* rel_type; // [R] node type of the relation's sources
    int d, H;
    __device__ __forceinline__ float scale(int x, int r, int h) const {
        return x ? 1.f : (mu ? weight(mu, (size_t)r * H + h) : 1.f) * rsqrtf((float)(d / H));
    }
};
struct Pair2 { void* p[2]; };

// Wbd[x][r][i][j] = c(r, h) * W[r][h][i % dh][j % dh] if i and j lie in the same head h, else 0.
template <typename T>
__global__ __launch_bounds__(256) void hgt_expand_kernel(int R, Halves<T> w, Pair2 Wbd) {
    const int x = blockIdx.y, d = w.d, dh = d / w.H;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)R * d * d) return;
    const int r = (int)(i / ((size_t)d * d)), a = (int)(i / d % d), b = (int)(i % d), h = a / dh;
    float v = 0.f;
    if (h == b / dh) v = w.scale(x, r, h) * weight(w.rel[x], (((size_t)r * w.H + h) * dh + a % dh) * dh + b % dh);
    static_cast<float*>(Wbd.p[x])[i] = v;
}

// One workgroup per (relation, head): dW[r][h] = c * block(dWbd[x][r], h); for the attention matrices also
// dmu[r][h] = sum(block .* W[r][h]) / sqrt(dh).
template <typename T>
__global__ __launch_bounds__(256) void hgt_extract_kernel(Halves<T> w, Pair2 dWbd, Pair2 dW, float* __restrict__ dmu) {
    __shared__ float red[256];
    const int x = blockIdx.y, d = w.d, H = w.H, r = blockIdx.x / H, h = blockIdx.x % H, dh = d / H;
    const float c = w.scale(x, r, h);
    float s = 0.f;
    for (int i = threadIdx.x; i < dh * dh; i += 256) {
        const float g = static_cast<const float*>(dWbd.p[x])[((size_t)r * d + h * dh + i / dh) * d + h * dh + i % dh];
        const size_t wi = ((size_t)r * H + h) * dh * dh + i;
        static_cast<float*>(dW.p[x])[wi] = c * g;
        s += g * weight(w.rel[x], wi);
    }
    if (x || !dmu) return;
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) dmu[r * H + h] = red[0] * rsqrtf((float)dh);
}

// Linear operator reordering (Ch.3 "Linear Operator Reordering": two linear operators in a row may be
// switched when that leaves a product between weights).  When every pair of a relation r has a source
// of one node type t(r), K[src] Watt[r] = X[src] (Wk[t(r)] Watt[r]): the per-pair key and message rows
// come straight from X with a folded per-relation weight, and K and V are never formed.
//   Wf[x][r][k][n] = c(r, h) * sum over j of Wnode[t(r)][k][h dh + j] * W[r][h][j][n % dh],  h the head of n
// stored as fp32 or rounded to bf16.
template <typename T, bool OUT16>
__global__ __launch_bounds__(256) void hgt_fold_kernel(int R, Halves<T> w, Pair2 Wf) {
    const int x = blockIdx.y, d = w.d, dh = d / w.H;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)R * d * d) return;
    const int r = (int)(i / ((size_t)d * d)), k = (int)(i / d % d), n = (int)(i % d), h = n / dh;
    const size_t wn = ((size_t)w.rel_type[r] * d + k) * d + h * dh, wr = ((size_t)r * w.H + h) * dh * dh + n % dh;
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;      // dh is a multiple of 16: four independent chains
#pragma unroll 4
    for (int j = 0; j < dh; j += 4) {
        s0 += weight(w.node[x], wn + j) * weight(w.rel[x], wr + (size_t)j * dh);
        s1 += weight(w.node[x], wn + j + 1) * weight(w.rel[x], wr + (size_t)(j + 1) * dh);
        s2 += weight(w.node[x], wn + j + 2) * weight(w.rel[x], wr + (size_t)(j + 2) * dh);
        s3 += weight(w.node[x], wn + j + 3) * weight(w.rel[x], wr + (size_t)(j + 3) * dh);
    }
    const float s = w.scale(x, r, h) * ((s0 + s1) + (s2 + s3));
    if (OUT16) static_cast<bf16_t*>(Wf.p[x])[i] = (bf16_t)(bf16_pack2(s, 0.f) & 0xFFFFu);
    else static_cast<float*>(Wf.p[x])[i] = s;
}

// Backward of the folding, from dWf[x] [R][d][d].  Two kinds of workgroups in one launch:
//   (r, h), the first R * H:  G = sum_k Wnode[t(r)][k][h dh + j] dWf[r][k][h dh + n];  dW[r][h] = c G,
//                             dmu[r][h] = sum(G .* W[r][h]) / sqrt(dh) (attention half)
//   (t, h, 32 rows k), the others:  dWnode[t][k][h dh + j] = sum over the relations r with t(r) = t, ascending, of
//                                   c(r, h) sum_n dWf[r][k][h dh + n] W[r][h][j][n]
// The operands of a step (32 rows of both) are staged in LDS; a thread forms DH * DH / 256 (or DH * 32 / 256) results, each in
// four chains over k mod 4, or in steps of four n (as one chain dWmsg at 300k edges, width 64, was
// 2.9e-7 off, 2.6e-7 so).  Both loops are unrolled as wholes: in steps of 4 and 8 they took 64 us for 50 (60 relations,
// heads of 32 columns) and 189 for 123 (heads of 64).
template <typename T, int DH>
__global__ __launch_bounds__(256) void hgt_fold_bwd_kernel(int R, Halves<T> w, Pair2 dWf_, Pair2 dW, Pair2 dWnode, float* __restrict__ dmu) {
    __shared__ float A[32][DH + 1], B[DH > 32 ? DH : 32][DH + 1], red[4];
    const int x = blockIdx.y, d = w.d, H = w.H, tid = threadIdx.x;
    const float* __restrict__ dWf = static_cast<const float*>(dWf_.p[x]);
    if ((int)blockIdx.x < R * H) {
        constexpr int NO = DH * DH / 256;
        const int r = blockIdx.x / H, h = blockIdx.x % H;
        const size_t wn = (size_t)w.rel_type[r] * d * d + h * DH, g0 = (size_t)r * d * d + h * DH;
        float part[NO][4], acc[NO];
#pragma unroll
        for (int q = 0; q < NO; ++q) part[q][0] = part[q][1] = part[q][2] = part[q][3] = 0.f;
        for (int k0 = 0; k0 < d; k0 += 32) {
            __syncthreads();
            for (int i = tid; i < 32 * DH; i += 256) {
                const size_t at = (size_t)(k0 + i / DH) * d + i % DH;
                A[i / DH][i % DH] = weight(w.node[x], wn + at);
                B[i / DH][i % DH] = dWf[g0 + at];
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 32; ++k)
#pragma unroll
                for (int q = 0; q < NO; ++q) part[q][k & 3] += A[k][(tid + 256 * q) / DH] * B[k][tid % DH];
        }
#pragma unroll
        for (int q = 0; q < NO; ++q) acc[q] = (part[q][0] + part[q][1]) + (part[q][2] + part[q][3]);
        const float c = w.scale(x, r, h);
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < NO; ++q) {
            const size_t wi = ((size_t)r * H + h) * DH * DH + tid + 256 * q;
            static_cast<float*>(dW.p[x])[wi] = c * acc[q];
            s += acc[q] * weight(w.rel[x], wi);
        }
        if (x || !dmu) return;
        s = group_sum<64>(s);
        if ((tid & 63) == 0) red[tid >> 6] = s;
        __syncthreads();
        if (tid == 0) dmu[r * H + h] = ((red[0] + red[1]) + (red[2] + red[3])) * rsqrtf((float)DH);
        return;
    }
    constexpr int NO = DH * 32 / 256;
    const int b = blockIdx.x - R * H, kt = d / 32;
    const int t = b / (H * kt), h = b / kt % H, k0 = b % kt * 32;
    float acc[NO];
#pragma unroll
    for (int q = 0; q < NO; ++q) acc[q] = 0.f;
    for (int r = 0; r < R; ++r) {
        if (w.rel_type[r] != t) continue;
        const float c = w.scale(x, r, h);
        __syncthreads();
        for (int i = tid; i < 32 * DH; i += 256) A[i / DH][i % DH] = dWf[(size_t)r * d * d + (size_t)(k0 + i / DH) * d + h * DH + i % DH];
        for (int i = tid; i < DH * DH; i += 256) B[i / DH][i % DH] = c * weight(w.rel[x], ((size_t)r * H + h) * DH * DH + i);
        __syncthreads();
        float p[NO];                              // one relation's sum first, then the relations in order
#pragma unroll
        for (int q = 0; q < NO; ++q) p[q] = 0.f;
#pragma unroll
        for (int n = 0; n < DH; n += 4)
#pragma unroll
            for (int q = 0; q < NO; ++q) {
                const float* const g = A[(tid + 256 * q) / DH] + n;
                const float* const wr = B[tid % DH] + n;
                p[q] += (g[0] * wr[0] + g[1] * wr[1]) + (g[2] * wr[2] + g[3] * wr[3]);
            }
#pragma unroll
        for (int q = 0; q < NO; ++q) acc[q] += p[q];
    }
#pragma unroll
    for (int q = 0; q < NO; ++q)
        static_cast<float*>(dWnode.p[x])[((size_t)t * d + k0 + (tid + 256 * q) / DH) * d + h * DH + tid % DH] = acc[q];
}

__global__ void add3_kernel(size_t n, const float* __restrict__ a, const float* __restrict__ b,
                            const float* __restrict__ c, float* __restrict__ out) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = a[i] + b[i] + c[i];
}

template <typename T>
Halves<T> halves(const HgtWeights& w) {
    auto p = [](const void* q) { return static_cast<const T*>(q); };
    return Halves<T>{{p(w.Wk), p(w.Wv)}, {p(w.Watt), p(w.Wmsg)}, p(w.mu), w.rel_type, w.d, w.H};
}

}  // namespace

// ---------------------------------------------------------------------------------------- launchers

rgnn_status_t hgt_expand(int R, const HgtWeights& w, float* Wbd_att, float* Wbd_msg, hipStream_t st) {
    KernelTimer kt(st, "hgt_expand");
    const dim3 grid(blocks_for((size_t)R * w.d * w.d, 256), 2);
    const Pair2 o{{Wbd_att, Wbd_msg}};
    if (w.bf16) hipLaunchKernelGGL(hgt_expand_kernel<bf16_t>, grid, dim3(256), 0, st, R, halves<bf16_t>(w), o);
    else hipLaunchKernelGGL(hgt_expand_kernel<float>, grid, dim3(256), 0, st, R, halves<float>(w), o);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}
rgnn_status_t hgt_extract(int R, const HgtWeights& w, float* dWbd_att, float* dWbd_msg, float* dWatt, float* dWmsg, float* dmu,
                          hipStream_t st) {
    KernelTimer kt(st, "hgt_extract");
    const Pair2 in{{dWbd_att, dWbd_msg}}, out{{dWatt, dWmsg}};
    if (w.bf16) hipLaunchKernelGGL(hgt_extract_kernel<bf16_t>, dim3(R * w.H, 2), dim3(256), 0, st, halves<bf16_t>(w), in, out, dmu);
    else hipLaunchKernelGGL(hgt_extract_kernel<float>, dim3(R * w.H, 2), dim3(256), 0, st, halves<float>(w), in, out, dmu);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}
rgnn_status_t hgt_fold(int R, const HgtWeights& w, void* Wf_att, void* Wf_msg, int out_bf16, hipStream_t st) {
    KernelTimer kt(st, "hgt_fold");
    const dim3 grid(blocks_for((size_t)R * w.d * w.d, 256), 2);
    const Pair2 o{{Wf_att, Wf_msg}};
    if (w.bf16 && out_bf16) hipLaunchKernelGGL((hgt_fold_kernel<bf16_t, true>), grid, dim3(256), 0, st, R, halves<bf16_t>(w), o);
    else if (w.bf16) hipLaunchKernelGGL((hgt_fold_kernel<bf16_t, false>), grid, dim3(256), 0, st, R, halves<bf16_t>(w), o);
    else if (!out_bf16) hipLaunchKernelGGL((hgt_fold_kernel<float, false>), grid, dim3(256), 0, st, R, halves<float>(w), o);
    else RGNN_FAIL(RGNN_EUNSUPPORTED, "hgt_fold: bf16 products are built for bf16 weights");
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}
rgnn_status_t hgt_fold_bwd(int T, int R, const HgtWeights& w, float* dWf_att, float* dWf_msg, float* dWk, float* dWv, float* dWatt,
                           float* dWmsg, float* dmu, hipStream_t st) {
    KernelTimer kt(st, "hgt_fold_bwd");
    const dim3 grid(R * w.H + T * w.H * (w.d / 32), 2);
    const Pair2 in{{dWf_att, dWf_msg}}, rel{{dWatt, dWmsg}}, node{{dWk, dWv}};
    const int dh = w.d / w.H;
#define RGNN_FOLD_BWD(DH_)                                                                                                      \
    do {                                                                                                                        \
        if (w.bf16) hipLaunchKernelGGL((hgt_fold_bwd_kernel<bf16_t, DH_>), grid, dim3(256), 0, st, R, halves<bf16_t>(w), in, rel, node, dmu); \
        else hipLaunchKernelGGL((hgt_fold_bwd_kernel<float, DH_>), grid, dim3(256), 0, st, R, halves<float>(w), in, rel, node, dmu);          \
    } while (0)
    if (dh == 16) RGNN_FOLD_BWD(16);
    else if (dh == 32) RGNN_FOLD_BWD(32);
    else if (dh == 64) RGNN_FOLD_BWD(64);
    else RGNN_FAIL(RGNN_EUNSUPPORTED, "hgt_fold_bwd: heads of 16, 32 or 64 columns, got %d", dh);
#undef RGNN_FOLD_BWD
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}
rgnn_status_t add3(size_t n, const float* a, const float* b, const float* c, float* out, hipStream_t st) {
    if (n == 0) return RGNN_OK;
    KernelTimer kt(st, "add3");
    hipLaunchKernelGGL(add3_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, st, n, a, b, c, out);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}

}  // namespace rgnn
