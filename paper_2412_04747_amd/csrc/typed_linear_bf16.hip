// Typed linear layer on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16), fp32 accumulation,
// for the bfloat16-input workloads:   Y[i] = A[g(i)] W[seg(i)]   where an operand or the result is fp32 or the width is below 128
// (all in bf16: typed_linear_fwd_bf16.hip; the backward: typed_linear_bwd_bf16.hip).
//
// Operands stored as bf16 (X, the given weights, and at width 128 every intermediate row
// tensor) go to the MFMA as they are, so their products are exact.  Operands that only exist
// in fp32 (the block-diagonal attention weights with mu/sqrt(dh) folded in; at widths below 128
// the intermediate rows) are split on the fly into two bf16 planes, x = hi + lo, and multiplied
// with two MFMAs, which keeps about 16 mantissa bits.  At these widths the kernel is bound by
// HBM traffic, not by the matrix cores, so the extra MFMAs are free.  The output rows are
// written as fp32 or rounded to bf16 (nearest even).
//
// Same wave-independent structure as the fp32 kernels: a workgroup keeps the segment's weight
// in LDS (as W_l[out column][contraction index], so a lane reads its B operand, eight
// consecutive contraction indices of one output column, as one 16-byte vector); each
// wavefront owns 32-row units, keeps the next unit's rows in flight in registers, and writes
// its accumulators straight to HBM.
#include "rgnn_internal.h"

namespace rgnn {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ int acc_row16(int v, int h) { return 8 * (v >> 2) + 4 * h + (v & 3); }

__device__ __forceinline__ void wave_lds_fence_b() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// fp32 -> bf16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ unsigned bf16_rne(float x) {
    unsigned u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}
// two fp32 -> packed bf16 pair (lo in bits 0..15), round to nearest even, one v_cvt_pk_bf16_f32
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned bf16_pack_rne(float lo, float hi) {
    const v2f v = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
// x = hi + lo (+ ~2^-17 |x|): both as bf16 bits
__device__ __forceinline__ void bf16_split(float x, unsigned& hi, unsigned& lo) {
    hi = bf16_rne(x);
    lo = bf16_rne(x - __uint_as_float(hi << 16));
}

struct TileArgsB {
    const int32_t* tile_seg;
    const int32_t* tile_row0;
    const int32_t* tile_row1;
    const int32_t* chunk_tile;
};

__device__ __forceinline__ int run_end_b(const int32_t* __restrict__ tile_seg, int ti, int t1) {
    const int seg = tile_seg[ti];
    int e = ti + 1;
    while (e < t1 && tile_seg[e] == seg) ++e;
    return e;
}

//   CD     contraction width, OD output width (both multiples of 32, CD a multiple of 16)
//   A_BF16 A rows are bf16 (exact) / fp32 (split)       W_BF16 weights are bf16 (exact) / fp32 (split)
//   GATHER rows are read through the gather list        SCATTER outputs are written through it as well
//   Y_BF16 output rows are stored as bf16 / fp32
// ldy: elements from one row of Y to the next.
template <int CD, int OD, bool A_BF16, bool W_BF16, bool GATHER, bool SCATTER, bool Y_BF16>
__global__ __launch_bounds__(256) void typed_linear_bf16_kernel(TileArgsB t, const void* __restrict__ Av,
                                                                const int32_t* __restrict__ gather,
                                                                const void* __restrict__ Wv, void* __restrict__ Yv, int ldy) {
    constexpr int NW = 4;
    constexpr int LS = CD + 8;                                // LDS row stride in bf16 elements (16-byte aligned rows)
    constexpr int OB = OD / 32;
    constexpr int APL = A_BF16 ? 1 : 2, WPL = W_BF16 ? 1 : 2; // planes (hi [, lo])
    constexpr int LPR = A_BF16 ? CD / 8 : CD / 4;             // lanes per A row (16-byte loads)
    constexpr int RPI = 64 / LPR, NX = 32 / RPI;
    extern __shared__ __align__(16) unsigned short lds[];
    unsigned short* Wl = lds;                                 // [WPL][OD][LS]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    unsigned short* Aw = lds + WPL * OD * LS + wave * (APL * 32 * LS + 64);   // [APL][32][LS] + 32 ints
    int* gidx = reinterpret_cast<int*>(Aw + APL * 32 * LS);
    const int m = lane & 31, kh = lane >> 5;
    const int ci = lane % LPR, ri = lane / LPR;
    const int t0 = t.chunk_tile[blockIdx.x], t1 = t.chunk_tile[blockIdx.x + 1];
    for (int ta = t0; ta < t1;) {
        const int tb = run_end_b(t.tile_seg, ta, t1);
        const int seg = t.tile_seg[ta];
        const int ra = t.tile_row0[ta], rbnd = t.tile_row1[tb - 1];
        const int nu = (rbnd - ra + 31) / 32;
        __syncthreads();                                      // every wavefront is done with the previous weight
        // weight of this segment into LDS as Wl[out column][contraction index]
        for (int i = tid; i < CD * OD; i += 64 * NW) {
            const int c = i / OD, o = i % OD;                 // contraction index, output column
            if (W_BF16) {
                Wl[o * LS + c] = static_cast<const unsigned short*>(Wv)[(size_t)seg * CD * OD + i];
            } else {
                unsigned hi, lo;
                bf16_split(static_cast<const float*>(Wv)[(size_t)seg * CD * OD + i], hi, lo);
                Wl[o * LS + c] = (unsigned short)hi;
                Wl[OD * LS + o * LS + c] = (unsigned short)lo;
            }
        }
        __syncthreads();
        v4u xr[NX];                                           // 16 bytes per load: 8 bf16 or 4 floats
        int gi[NX], gcur[NX];
#define RGNN_FETCH_IDX(U)                                                       \
    _Pragma("unroll") for (int it = 0; it < NX; ++it) {                         \
        const int row_ = min(ra + (U) * 32 + ri + it * RPI, rbnd - 1);          \
        gi[it] = GATHER ? gather[row_] : row_;                                  \
    }
#define RGNN_FETCH_ROWS()                                                       \
    _Pragma("unroll") for (int it = 0; it < NX; ++it) {                         \
        const char* p_ = static_cast<const char*>(Av) + (size_t)gi[it] * CD * (A_BF16 ? 2 : 4) + ci * 16; \
        xr[it] = *reinterpret_cast<const v4u*>(p_);                             \
        gcur[it] = gi[it];                                                      \
    }
        RGNN_FETCH_IDX(wave)
        RGNN_FETCH_ROWS()
        RGNN_FETCH_IDX(wave + NW)
        for (int u = wave; u < nu; u += NW) {
#pragma unroll
            for (int it = 0; it < NX; ++it) {
                const int r = ri + it * RPI;
                if (A_BF16) {
                    *reinterpret_cast<v4u*>(Aw + r * LS + ci * 8) = xr[it];
                } else {
                    unsigned h[4], l[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) bf16_split(__uint_as_float(xr[it][e]), h[e], l[e]);
                    uint2 hv = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
                    uint2 lv = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
                    *reinterpret_cast<uint2*>(Aw + r * LS + ci * 4) = hv;
                    *reinterpret_cast<uint2*>(Aw + 32 * LS + r * LS + ci * 4) = lv;
                }
                if (SCATTER && ci == 0) gidx[r] = gcur[it];
            }
            wave_lds_fence_b();
            RGNN_FETCH_ROWS()             // unit u + NW
            RGNN_FETCH_IDX(u + 2 * NW)
            v16f acc[OB];
#pragma unroll
            for (int b = 0; b < OB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
#pragma unroll 2
            for (int s = 0; s < CD / 16; ++s) {
                const int c0 = 16 * s + 8 * kh;
                const bf16x8 ah = *reinterpret_cast<const bf16x8*>(Aw + m * LS + c0);
                bf16x8 al;
                if (!A_BF16) al = *reinterpret_cast<const bf16x8*>(Aw + 32 * LS + m * LS + c0);
#pragma unroll
                for (int b = 0; b < OB; ++b) {
                    const bf16x8 bh = *reinterpret_cast<const bf16x8*>(Wl + (b * 32 + m) * LS + c0);
                    acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc[b], 0, 0, 0);
                    if (!A_BF16) acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, acc[b], 0, 0, 0);
                    if (!W_BF16) {
                        const bf16x8 bl = *reinterpret_cast<const bf16x8*>(Wl + OD * LS + (b * 32 + m) * LS + c0);
                        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, acc[b], 0, 0, 0);
                    }
                }
            }
            const int rows_left = rbnd - (ra + u * 32);
            if (!Y_BF16) {
                // accumulators straight to HBM: lanes 0..31 and 32..63 each write one 128-byte line
                float* __restrict__ Y = static_cast<float*>(Yv);
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int r = acc_row16(v, kh);
                    if (r < rows_left) {
                        const size_t d = SCATTER ? (size_t)gidx[r] : (size_t)(ra + u * 32 + r);
#pragma unroll
                        for (int b = 0; b < OB; ++b) Y[d * ldy + b * 32 + m] = acc[b][v];
                    }
                }
            } else {
                // bf16 rows go through the wavefront's A area of LDS (free once the operand reads are
                // done), so that HBM sees whole rows: registers v and v + 1 hold rows r and r + 1 of
                // column m; neighbouring lanes swap one of the two, an even lane then owns (row r;
                // columns m, m + 1), an odd lane (row r + 1; columns m - 1, m), and each writes one
                // packed pair.  Then 16-byte pieces of whole rows are copied out, OD / 8 lanes per row.
                static_assert(!Y_BF16 || (A_BF16 && OD <= CD), "the output tile is staged in the A area");
                unsigned short* __restrict__ Y = static_cast<unsigned short*>(Yv);
                const bool odd = m & 1;
                wave_lds_fence_b();
#pragma unroll
                for (int v = 0; v < 16; v += 2) {
                    const int r = acc_row16(v, kh) + (odd ? 1 : 0);
#pragma unroll
                    for (int b = 0; b < OB; ++b) {
                        // quad_perm [1, 0, 3, 2]: the neighbouring lane's two values
                        const float a0 = acc[b][v], a1 = acc[b][v + 1];
                        const float n0 = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(a0), 0xB1, 0xF, 0xF, true));
                        const float n1 = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(a1), 0xB1, 0xF, 0xF, true));
                        const unsigned w = bf16_pack_rne(odd ? n1 : a0, odd ? a1 : n0);
                        *reinterpret_cast<unsigned*>(Aw + r * LS + b * 32 + (m & ~1)) = w;
                    }
                }
                wave_lds_fence_b();
                constexpr int LPO = OD / 8, RPP = 64 / LPO;       // lanes per output row, rows per pass
                const int oc = lane % LPO, orow = lane / LPO;
#pragma unroll
                for (int pass = 0; pass < 32 / RPP; ++pass) {
                    const int r = orow + pass * RPP;
                    if (r < rows_left) {
                        const size_t d = SCATTER ? (size_t)gidx[r] : (size_t)(ra + u * 32 + r);
                        __builtin_nontemporal_store(*reinterpret_cast<const v4u*>(Aw + r * LS + oc * 8), reinterpret_cast<v4u*>(Y + d * ldy + oc * 8));
                    }
                }
            }
            wave_lds_fence_b();           // operand reads (and gidx reads) are done before the next unit's rows land
        }
#undef RGNN_FETCH_IDX
#undef RGNN_FETCH_ROWS
        ta = tb;
    }
}

template <int CD, int OD, bool A_BF16, bool W_BF16, bool GATHER, bool SCATTER, bool Y_BF16>
static rgnn_status_t launch(const TypedLinearBf16Args& a, hipStream_t st) {
    constexpr int LS = CD + 8, APL = A_BF16 ? 1 : 2, WPL = W_BF16 ? 1 : 2;
    const size_t lds = sizeof(unsigned short) * ((size_t)WPL * OD * LS + 4 * (APL * 32 * LS + 64));
    auto kern = typed_linear_bf16_kernel<CD, OD, A_BF16, W_BF16, GATHER, SCATTER, Y_BF16>;
    RGNN_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds));
    KernelTimer kt(st, a.label ? a.label : "typed_linear_bf16");
    TileArgsB t{a.tiles->tile_seg, a.tiles->tile_row0, a.tiles->tile_row1, a.tiles->chunk_tile};
    hipLaunchKernelGGL(kern, dim3(a.tiles->num_chunks), dim3(256), lds, st, t, a.A, a.gather, a.W, a.Y, a.y_stride * OD);
    RGNN_HIP(hipGetLastError());
    return RGNN_OK;
}

template <int D, bool A_BF16, bool W_BF16, bool Y_BF16>
static rgnn_status_t launch_gs(const TypedLinearBf16Args& a, hipStream_t st) {
    const bool g = a.gather != nullptr, sc = g && a.scatter_out;
    if (g && sc) return launch<D, D, A_BF16, W_BF16, true, true, Y_BF16>(a, st);
    if (g) return launch<D, D, A_BF16, W_BF16, true, false, Y_BF16>(a, st);
    return launch<D, D, A_BF16, W_BF16, false, false, Y_BF16>(a, st);
}

// The combinations the layers use.  Below width 128 only products with fp32 results occur (intermediate rows are
// fp32 there); at width 128 every row operand is bf16.
template <int D>
static rgnn_status_t launch_d(const TypedLinearBf16Args& a, hipStream_t st) {
    if constexpr (D < 128) {
        if (a.y_bf16) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_bf16: combination needs width 128");
        if (a.a_bf16 && a.w_bf16) return launch_gs<D, true, true, false>(a, st);      // X W
        if (!a.a_bf16 && a.w_bf16) return launch_gs<D, false, true, false>(a, st);    // Z Wo
        if (!a.a_bf16 && !a.w_bf16) return launch_gs<D, false, false, false>(a, st);  // K Watt_bd
    } else {
        if (!a.a_bf16) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_bf16: width 128 takes bf16 rows");
        if (a.w_bf16 && !a.y_bf16) return launch_gs<D, true, true, false>(a, st);  // Z Wo -> out
        if (!a.w_bf16 && a.y_bf16) return launch_gs<D, true, false, true>(a, st);  // K Watt_bd -> Ka
    }
    RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_bf16: operand combination not built");
}

rgnn_status_t typed_linear_bf16(int d, const TypedLinearBf16Args& a, hipStream_t st) {
    if (a.tiles->num_tiles == 0) return RGNN_OK;
    if (d == 128) return launch_d<128>(a, st);
    if (d == 64) return launch_d<64>(a, st);
    if (d == 32) return launch_d<32>(a, st);
    RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_bf16: width %d not supported (32/64/128)", d);
}

}  // namespace rgnn
