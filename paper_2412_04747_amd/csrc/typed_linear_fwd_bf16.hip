// Forward of the typed linear layer with input rows, weights and result rows in bf16, width 128 (v_mfma_f32_32x32x16_bf16, fp32 accumulation):
//   Y[i] = X[g(i)] W[seg(i)]                              one weight, rows in order or scattered back through the gather list
//   Y[i] = (X[g(i)] W0[seg(i)], X[g(i)] W1[seg(i)])       two weights, side by side, 512 bytes per row (HGT's key and message)
//
// Bound by HBM.  With two weights a row is gathered once and its results leave as one row: 5.4M pairs 0.75 ms (4.1 GB, 5.5 TB/s); as two
// products, which gathered the input rows twice and wrote the result rows in halves, 1.07 ms.  With one weight, against one
// unit of 32 rows per wavefront (typed_linear_bf16.hip): 200k nodes scattered back 30 us for 38, 2M nodes 235 for 234, 14.5M pairs
// 1347 for 1349.  (fp32 result rows stay there: from this layout they leave in 16-byte pieces, 334 us for 286 at 2M nodes.)
//
// A workgroup of eight wavefronts takes a chunk of 64-row tiles.  A tile's rows are brought to registers one tile ahead and written to
// LDS row-major, swizzled as in the backward (typed_linear_bwd_bf16.hip); the weights lie there as they are in memory, and their
// operand (eight consecutive input features of an output feature) comes through the transposing LDS read.  Each wavefront forms 32 rows
// x 32 output features of every product; bf16 results are packed into a tile in LDS, whose rows leave in 16-byte pieces.
#include "rgnn_internal.h"
#include "device_utils.h"

namespace rgnn {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

struct FwdArgs {
    const int32_t* tile_seg;
    const int32_t* tile_row0;
    const int32_t* tile_row1;
    const int32_t* chunk_tile;
    const bf16_t* X;
    const int32_t* gather;
    const bf16_t* W[2];
    void* Y;
};


constexpr int D = 128, TILE = 64 * 2 * D, WT = D * 2 * D;      // bytes of 64 rows and of a weight

//   NB  weights      SCATTER  row i of the result goes where row i of the input came from
template <int NB, bool SCATTER>
__device__ __forceinline__ void fwd_tiles(const FwdArgs& a) {
    static_assert(NB == 1 || !SCATTER, "combinations the layers use");
    extern __shared__ __align__(16) unsigned char lds[];
    unsigned char* const Wl = lds;                        // [NB][128][256]
    unsigned char* const Xt = lds + NB * WT;              // [64][256]
    unsigned char* const St = Xt + TILE;                  // [NB][64][256]  the result rows on their way out
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = lane & 31, kh = lane >> 5;
    // rows in and out: 16 lanes per 256 bytes, two rows per thread (in), four pieces (out)
    const int lc = tid & 15, lr = tid >> 4;
    const int io = lr * 256 + ((lc ^ swz(lr)) << 4);
    // this wavefront's block: 32 rows x output features 16 fb + (0..15) and 64 further, of both weights
    const int fb = wave & 3, rb = wave >> 2;
    const int ti16 = lane & 15, tg = (lane >> 4) & 1;
    int woff[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int r = 8 * kh + 4 * t + (ti16 >> 2), piece = (ti16 & 3) >> 1, half = (ti16 & 1) * 8;
        woff[t] = r * 256 + (((2 * (fb + 4 * tg) + piece) ^ swz(r)) << 4) + half;
    }
    const int xrow = (rb * 32 + m) * 256, xsw = (kh ^ swz(m)) << 4;
    const int t0 = a.chunk_tile[blockIdx.x], t1 = a.chunk_tile[blockIdx.x + 1];
    if (t0 >= t1) return;
    rgnn_v4u xr[2];
    int gi[2], gcur[2];
    TileTable tt(a.tile_seg, a.tile_row0, a.tile_row1, t0, t1);
    auto fetch_idx = [&](int ti) {
        const int l = tt.lane_of(ti), row0 = tt.row0_at(l), row1 = tt.row1_at(l);
#pragma unroll
        for (int k = 0; k < 2; ++k) gi[k] = a.gather[min(row0 + lr + 32 * k, row1 - 1)];
    };
    auto fetch = [&]() {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            xr[k] = *reinterpret_cast<const rgnn_v4u*>(a.X + (size_t)gi[k] * D + lc * 8);
            gcur[k] = gi[k];
        }
    };
    fetch_idx(t0);
    fetch();
    fetch_idx(min(t0 + 1, t1 - 1));
    int cur_seg = -1;
    for (int ti = t0; ti < t1; ++ti) {
        const int tl = tt.lane_of(ti), seg = tt.seg_at(tl);
        if (seg != cur_seg) {              // (all operand reads of the previous tile lie before its second barrier)
            cur_seg = seg;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    *reinterpret_cast<rgnn_v4u*>(Wl + nb * WT + io + k * 32 * 256) =
                        *reinterpret_cast<const rgnn_v4u*>(a.W[nb] + (size_t)seg * D * D + (size_t)(lr + 32 * k) * D + lc * 8);
        }
        const int row0 = tt.row0_at(tl), rows = tt.row1_at(tl) - row0;
        int gout[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            *reinterpret_cast<rgnn_v4u*>(Xt + io + k * 32 * 256) = xr[k];   // past the end the last row again: not stored
            gout[k] = gcur[k];
        }
        __syncthreads();   // the tile is complete, and the previous one's result rows have been read out
        fetch();           // unconditional, past the end the last tile again: see the backward
        fetch_idx(min(ti + 2, t1 - 1));
        v16f d[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) d[nb][v] = 0.f;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const bf16x8 bx = *reinterpret_cast<const bf16x8*>(Xt + xrow + (xsw ^ (s << 5)));
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const unsigned char* w = Wl + nb * WT + s * 4096;
                d[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr8(w + woff[0], w + woff[1]), bx, d[nb], 0, 0, 0);
            }
        }
        // d[v] = row rb * 32 + m, block row 8 (v / 4) + 4 kh + v % 4: features 16 fb + (0..15), then 64 further
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int piece = 2 * fb + (q & 1) + 8 * (q >> 1);
                *reinterpret_cast<uint2*>(St + nb * TILE + xrow + ((piece ^ swz(m)) << 4) + 8 * kh) =
                    make_uint2(bf16_pack2(d[nb][4 * q], d[nb][4 * q + 1]), bf16_pack2(d[nb][4 * q + 2], d[nb][4 * q + 3]));
            }
        __syncthreads();   // operand reads are done, the result tile is complete
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int r = lr + 32 * k;
                const size_t to = SCATTER ? (size_t)gout[k] : (size_t)(row0 + r);
                if (r < rows)
                    __builtin_nontemporal_store(*reinterpret_cast<const rgnn_v4u*>(St + nb * TILE + io + k * 32 * 256),
                                                reinterpret_cast<rgnn_v4u*>(static_cast<bf16_t*>(a.Y) + (to * NB + nb) * D + lc * 8));
            }
    }
}

// One weight: two workgroups per compute unit; two weights take the room of both.
template <bool SCATTER>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4))) void typed_linear_fwd_bf16_kernel(FwdArgs a) { fwd_tiles<1, SCATTER>(a); }
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void typed_linear_fwd_bf16_two_kernel(FwdArgs a) { fwd_tiles<2, false>(a); }

}  // namespace

rgnn_status_t typed_linear_fwd_bf16(const TypedLinearFwdBf16Args& x, hipStream_t st) {
    const TileList& t = *x.tiles;
    if (t.num_tiles == 0) return RGNN_OK;
    if (!x.gather || (x.W2 && x.scatter_out)) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_fwd_bf16: gathered rows; two weights with result rows in order only");
    const int nb = x.W2 ? 2 : 1;
    const size_t lds = (size_t)nb * WT + (1 + nb) * TILE;
    const FwdArgs a{t.tile_seg, t.tile_row0, t.tile_row1, t.chunk_tile, static_cast<const bf16_t*>(x.X), x.gather,
                    {static_cast<const bf16_t*>(x.W), static_cast<const bf16_t*>(x.W2)}, x.Y};
    auto kern = x.W2 ? typed_linear_fwd_bf16_two_kernel : x.scatter_out ? typed_linear_fwd_bf16_kernel<true> : typed_linear_fwd_bf16_kernel<false>;
    RGNN_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds));
    KernelTimer kt(st, x.label);
    hipLaunchKernelGGL(kern, dim3(t.num_chunks), dim3(512), lds, st, a);
    RGNN_HIP(hipGetLastError());
    return RGNN_OK;
}

}  // namespace rgnn
