// Weight kernels of the HGT layer: block-diagonal expansion of the per-(relation, head) matrices, folding of the node
// linears into them, and their backward.  (Caption of the thesis figure "HGT and RGAT layer": attention of HGT is an
// edgewise dot product between the relation-transformed key of the source and the query of the destination; the message
// depends only on (source node, edge type), so both are stored once per pair.  The edge walks are in hgt_walk.hip.)
//
// The d_head x d_head matrices W[r][h] are expanded to one block-diagonal d x d matrix per
// relation so that the relation-segmented typed-linear kernel serves them unchanged; with
// bf16 or fp32 inputs that kernel is bound by HBM traffic at these widths, so the extra
// zero blocks cost no time.
#include "rgnn_internal.h"
#include "traversal.h"
#include "device_utils.h"

namespace rgnn {

// Wbd[r][i][j] = c(r, h) * W[r][h][i % dh][j % dh] if i and j lie in the same head h, else 0.
// c = (mu ? mu[r][h] : 1) / sqrt(dh) when `scaled` (attention), 1 otherwise (message).
__global__ void hgt_expand_kernel(int R, int d, int H, const float* __restrict__ W, const float* __restrict__ mu,
                                  int scaled, float* __restrict__ Wbd) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t total = (size_t)R * d * d;
    if (i >= total) return;
    const int dh = d / H;
    const int r = (int)(i / ((size_t)d * d)), a = (int)(i / d % d), b = (int)(i % d);
    const int ha = a / dh, hb = b / dh;
    float v = 0.f;
    if (ha == hb) {
        float c = 1.f;
        if (scaled) c = (mu ? mu[r * H + ha] : 1.f) * rsqrtf((float)dh);
        v = c * W[(((size_t)r * H + ha) * dh + a % dh) * dh + b % dh];
    }
    Wbd[i] = v;
}

// One workgroup per (relation, head): dW[r][h] = c * block(dWbd[r], h); for the attention
// matrices also dmu[r][h] = sum(block .* W[r][h]) / sqrt(dh).
__global__ void hgt_extract_kernel(int d, int H, const float* __restrict__ dWbd, const float* __restrict__ W,
                                   const float* __restrict__ mu, int scaled, float* __restrict__ dW,
                                   float* __restrict__ dmu) {
    __shared__ float red[256];
    const int r = blockIdx.x / H, h = blockIdx.x % H, dh = d / H;
    const float inv = rsqrtf((float)dh);
    const float c = scaled ? (mu ? mu[r * H + h] : 1.f) * inv : 1.f;
    float s = 0.f;
    for (int i = threadIdx.x; i < dh * dh; i += blockDim.x) {
        const int a = i / dh, b = i % dh;
        const float g = dWbd[((size_t)r * d + h * dh + a) * d + h * dh + b];
        const size_t wi = ((size_t)r * H + h) * dh * dh + i;
        dW[wi] = c * g;
        s += g * W[wi];
    }
    if (!(scaled && dmu)) return;
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) dmu[r * H + h] = red[0] * inv;
}

// Linear operator reordering (Ch.3 "Linear Operator Reordering": two linear operators in a row may be
// switched when that leaves a product between weights).  When every pair of a relation r has a source
// of one node type t(r), K[src] Watt[r] = X[src] (Wk[t(r)] Watt[r]): the per-pair key and message rows
// come straight from X with a folded per-relation weight, and K and V are never formed.
//   Wf[r][k][n] = sum over j in the head of n of Wnode[t(r)][k][j] * Wbd[r][j][n]
// Written as fp32 (Wf) or rounded to bf16 (Wf16), whichever is given.
__global__ void hgt_fold_kernel(int R, int d, int H, const int32_t* __restrict__ rel_type,
                                const float* __restrict__ Wnode, const float* __restrict__ Wbd, float* __restrict__ Wf,
                                bf16_t* __restrict__ Wf16) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)R * d * d) return;
    const int dh = d / H;
    const int r = (int)(i / ((size_t)d * d)), k = (int)(i / d % d), n = (int)(i % d);
    const float* Wn = Wnode + ((size_t)rel_type[r] * d + k) * d;
    const float* Wb = Wbd + (size_t)r * d * d;
    const int j0 = n / dh * dh;
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;      // dh is a multiple of 16: four independent chains
#pragma unroll 2
    for (int j = j0; j < j0 + dh; j += 4) {
        const float4 w4 = *reinterpret_cast<const float4*>(Wn + j);
        s0 += w4.x * Wb[(size_t)j * d + n];
        s1 += w4.y * Wb[(size_t)(j + 1) * d + n];
        s2 += w4.z * Wb[(size_t)(j + 2) * d + n];
        s3 += w4.w * Wb[(size_t)(j + 3) * d + n];
    }
    const float s = (s0 + s1) + (s2 + s3);
    if (Wf) Wf[i] = s;
    if (Wf16) Wf16[i] = (bf16_t)(bf16_pack2(s, 0.f) & 0xFFFFu);
}

// dWbd[r][j][n] = sum_k Wnode[t(r)][k][j] * dWf[r][k][n] for j, n in the same head (other entries are not written)
__global__ void hgt_fold_bwd_rel_kernel(int R, int d, int H, const int32_t* __restrict__ rel_type,
                                        const float* __restrict__ Wnode, const float* __restrict__ dWf,
                                        float* __restrict__ dWbd) {
    const int dh = d / H;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;    // (r, j, n') with n' inside the head of j
    if (i >= (size_t)R * d * dh) return;
    const int r = (int)(i / ((size_t)d * dh)), j = (int)(i / dh % d), n = j / dh * dh + (int)(i % dh);
    const float* Wn = Wnode + (size_t)rel_type[r] * d * d;
    const float* G = dWf + (size_t)r * d * d;
    // four partial sums over k = 4 i + q keep eight independent loads in flight (d is a multiple of 32)
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
#pragma unroll 2
    for (int k = 0; k < d; k += 4) {
        s0 += Wn[(size_t)k * d + j] * G[(size_t)k * d + n];
        s1 += Wn[(size_t)(k + 1) * d + j] * G[(size_t)(k + 1) * d + n];
        s2 += Wn[(size_t)(k + 2) * d + j] * G[(size_t)(k + 2) * d + n];
        s3 += Wn[(size_t)(k + 3) * d + j] * G[(size_t)(k + 3) * d + n];
    }
    dWbd[((size_t)r * d + j) * d + n] = (s0 + s1) + (s2 + s3);
}

// dWnode[t][k][j] = sum over relations r with t(r) = t, ascending, of sum over n in the head of j of dWf[r][k][n] * Wbd[r][j][n]
__global__ void hgt_fold_bwd_node_kernel(int T, int R, int d, int H, const int32_t* __restrict__ rel_type,
                                         const float* __restrict__ Wbd, const float* __restrict__ dWf,
                                         float* __restrict__ dWnode) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)T * d * d) return;
    const int dh = d / H;
    const int t = (int)(i / ((size_t)d * d)), k = (int)(i / d % d), j = (int)(i % d);
    const int n0 = j / dh * dh;
    float s = 0.f;
    for (int r = 0; r < R; ++r) {
        if (rel_type[r] != t) continue;
        const float* G = dWf + ((size_t)r * d + k) * d;
        const float* Wb = Wbd + ((size_t)r * d + j) * d;
        float p = 0.f;     // dh is a multiple of 16 and n0 of dh: 16-byte loads
        for (int n = n0; n < n0 + dh; n += 4) {
            const float4 gv = *reinterpret_cast<const float4*>(G + n), wv = *reinterpret_cast<const float4*>(Wb + n);
            p += (gv.x * wv.x + gv.y * wv.y) + (gv.z * wv.z + gv.w * wv.w);
        }
        s += p;
    }
    dWnode[i] = s;
}

__global__ void add3_kernel(size_t n, const float* __restrict__ a, const float* __restrict__ b,
                            const float* __restrict__ c, float* __restrict__ out) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = a[i] + b[i] + c[i];
}

// ---------------------------------------------------------------------------------------- launchers

rgnn_status_t hgt_expand(int R, int d, int H, const float* W, const float* mu, int scaled, float* Wbd, hipStream_t st) {
    KernelTimer kt(st, "hgt_expand");
    hipLaunchKernelGGL(hgt_expand_kernel, dim3(blocks_for((size_t)R * d * d, 256)), dim3(256), 0, st, R, d, H, W, mu,
                       scaled, Wbd);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}
rgnn_status_t hgt_extract(int R, int d, int H, const float* dWbd, const float* W, const float* mu, int scaled, float* dW,
                          float* dmu, hipStream_t st) {
    KernelTimer kt(st, "hgt_extract");
    hipLaunchKernelGGL(hgt_extract_kernel, dim3(R * H), dim3(256), 0, st, d, H, dWbd, W, mu, scaled, dW, dmu);
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}
rgnn_status_t hgt_fold(int R, int d, int H, const int32_t* rel_type, const float* Wnode, const float* Wbd, float* Wf,
                       void* Wf16, hipStream_t st) {
    KernelTimer kt(st, "hgt_fold");
    hipLaunchKernelGGL(hgt_fold_kernel, dim3(blocks_for((size_t)R * d * d, 256)), dim3(256), 0, st, R, d, H, rel_type, Wnode,
                       Wbd, Wf, static_cast<bf16_t*>(Wf16));
    RGNN_CHECK_LAUNCH();
    return RGNN_OK;
}
rgnn_status_t hgt_fold_bwd(int T, int R, int d, int H, const int32_t* rel_type, const float* Wnode, const float* Wbd,
                           const float* dWf, float* dWbd, float* dWnode, hipStream_t st) {
    KernelTimer kt(st, "hgt_fold_bwd");
    hipLaunchKernelGGL(hgt_fold_bwd_rel_kernel, dim3(blocks_for((size_t)R * d * (d / H), 256)), dim3(256), 0, st, R, d, H,
                       rel_type, Wnode, dWf, dWbd);
    RGNN_CHECK_LAUNCH();
    hipLaunchKernelGGL(hgt_fold_bwd_node_kernel, dim3(blocks_for((size_t)T * d * d, 256)), dim3(256), 0, st, T, R, d, H,
                       rel_type, Wbd, dWf, dWnode);
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
