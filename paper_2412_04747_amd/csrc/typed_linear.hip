// Relation-segmented typed linear layer on the fp32 matrix cores, widths 32 and 64 (width 128: typed_linear_split.hip,
// and the forward here where the sign of its result matters).
//
// Forward   Y[i] = X[gather[i]] W[seg(i)]          (thesis Ch.3: segment MM, Y[S] = X[G] x W[T];
//                                                   rows are presorted by type so one weight serves a segment)
// Backward  dXrow[i] = dY[i] W[seg(i)]^T,  dW[s] = sum_{i in s} X[gather[i]]^T dY[i]
//
// Rows are cut into 64-row tiles that never straddle a segment; a persistent workgroup
// walks a contiguous chunk of tiles and keeps the current segment's weight in LDS,
// reloading it only when the segment changes.  The products run on v_mfma_f32_32x32x2_f32.  The K index of the MFMA is a free permutation, so each lane
// reads its A operand as 16-byte LDS vectors: lane (m, half) owns k = half*K/2 + 0..K/2-1.
#include "rgnn_internal.h"
#include "device_utils.h"

#include <algorithm>

namespace rgnn {

typedef float v16f __attribute__((ext_vector_type(16)));
// Native 4-float vector for the register prefetch buffers: unlike HIP's float4 struct it is
// copied with plain vector loads and stores, so arrays of it stay in registers.
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v16f mfma32(float a, float b, v16f c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Row of the 32x32 accumulator held in register v of a lane in half `h` (lane / 32);
// the column is lane % 32.
__device__ __forceinline__ int acc_row(int v, int h) { return 8 * (v >> 2) + 4 * h + (v & 3); }

struct TileArgs {
    const int32_t* tile_seg;
    const int32_t* tile_row0;
    const int32_t* tile_row1;
    const int32_t* chunk_tile;
    const int32_t* chunk_slot;
};

// ---------------------------------------------------------------------------------------
// Wave-independent kernels (feature widths up to 64).
//
// Within a run of tiles that share a segment, the wavefronts of a workgroup do not
// synchronise with each other: wavefront w owns the 32-row units w, w + NW, ... of the run,
// stages them in its private LDS region and keeps the rows of its next unit in flight in
// registers (the gather indices one unit further ahead).  Workgroup barriers are needed only
// when the segment changes (reload of the shared weight tile, flush of the weight-gradient
// partial sums).  This keeps 8 KB (forward) / 16 KB (backward) of HBM reads in flight per
// wavefront at all times, which is what the random row gather needs.
//
// LDS accesses of one wavefront are executed in issue order, so inside a wavefront a store
// followed by a load of another lane's data needs no barrier; wave_lds_fence() only stops
// the compiler from moving LDS accesses across it and waits for outstanding LDS operations.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// First tile index >= ti whose segment differs from tile ti's (or t1): 64 tiles per step (one after the other they cost a chunk
// of 149 tiles some 5 us before its first row).
__device__ __forceinline__ int run_end(const int32_t* __restrict__ tile_seg, int ti, int t1, int lane) {
    const int seg = tile_seg[ti];
    if (tile_seg[t1 - 1] == seg) return t1;              // (tiles lie in segment order) the usual case of a short chunk
    for (int e = ti; e < t1; e += 64) {
        const unsigned long long other = __ballot(tile_seg[min(e + lane, t1 - 1)] != seg);
        if (other) return e + __builtin_ctzll(other);
    }
    return t1;
}

// Compile-time switches of the wave kernels.  They are template parameters rather than
// run-time flags so that the unit loop holds no conditional global load: with one, the
// compiler has to wait for every outstanding memory operation (the prefetched rows and the
// previous unit's stores) at each use.
//   GATHER   rows are read through the gather list        SCATTER  outputs are written through it as well
//   ACCUM    forward: Y += result (relu: then max(Y, 0))  VEC      forward: s_out = Y_row . vec[seg], per head:
//                                                                  s_out[row][h] over the h-th of s_heads column slices
//   DYG      backward: dY rows are read through the list  RS       backward: rowscale / Avec / xvec in use
//   OS       the rows of Y are OS * ND floats apart (2: the key or message half of HGT's pair rows)
//   XSEL     input rows come from two tensors: list entry g >= 0 is row g of X, otherwise row g & 0x7FFFFFFF of X2 (the rows
//            per run: a run's only source, or the sum of its sources); forward: row i of the result goes to row to[i] of Y
//
// At width 128 the stage holds half of the columns at a time, so that eight wavefronts fit beside the 64 KB weight: two per
// SIMD, one multiplying while the other stages; and the result goes to memory straight from the accumulators, a 128-byte line
// of two rows per store.  (Four wavefronts with whole rows, result through the stage: 235 us for 702k pairs, now 205; 977 us for
// 2.46M pairs of 500 relations, now 785.)  At 64 x 64, where the rows' bytes bound the kernel, direct stores take 186 us
// for the 175 of whole 256-byte rows through the stage (2.1M pairs); from 32 to 64 columns 120 for 130, but 40 for 38 where
// the rows of Y are read first (300k rows).
template <int KD, int ND, bool VEC, bool ACCUM>
struct FwdShape {
    static constexpr bool HALVES = KD == 128 && !VEC;
    static constexpr int NW = HALVES ? 8 : 4;               // wavefronts per workgroup
    static constexpr int KS = HALVES ? KD / 2 : KD;         // columns in the stage
    static constexpr bool DIRECT = HALVES || (KD < ND && !VEC && !ACCUM);   // result straight from the accumulators
    static constexpr int XS = (!DIRECT && ND > KS ? ND : KS) + 4;   // row stride of the per-wave stage
    static constexpr size_t LDS = sizeof(float) * (KD * ND + NW * 32 * XS);
};
// what lane r keeps for the lower half of the wavefront, lane r + 4 for the upper one
__device__ __forceinline__ int row_of_half(int v, int r, int kh) {
    const int a = __builtin_amdgcn_readlane(v, r), b = __builtin_amdgcn_readlane(v, r + 4);
    return kh ? b : a;
}
// row g of X, or with XSEL of the tensor that g's top bit says
template <int D, bool XSEL>
__device__ __forceinline__ const float* input_row(const float* __restrict__ X, const float* __restrict__ X2, int g) {
    return (XSEL && g < 0 ? X2 : X) + (size_t)(XSEL ? g & 0x7FFFFFFF : g) * D;
}
template <int KD, int ND, bool GATHER, bool SCATTER, bool ACCUM, bool VEC, int OS = 1, bool XSEL = false>
__device__ __forceinline__ void fwd_wave(const TileArgs& t, int chunk, const float* __restrict__ X, const int32_t* __restrict__ gather,
                                         const float* __restrict__ W, float* __restrict__ Y, const float* __restrict__ vec,
                                         float* __restrict__ s_out, int s_heads, int relu, const float* __restrict__ X2 = nullptr,
                                         const int32_t* __restrict__ to = nullptr) {
    static_assert(!XSEL || (GATHER && !SCATTER && !ACCUM && !VEC), "two input tensors: plain products of gathered rows");
    using S = FwdShape<KD, ND, VEC, ACCUM>;
    constexpr int NW = S::NW, XS = S::XS, KS = S::KS, PH = KD / KS;
    constexpr int CB = ND / 32;
    constexpr bool DIRECT = S::DIRECT;
    constexpr int LPRI = KD / 4, RPI = 64 / LPRI, NX = 32 / RPI;   // input: lanes per row, rows per load, loads per unit
    constexpr int LPRO = ND / 4, RPO = 64 / LPRO, NO = 32 / RPO;
    static_assert(!SCATTER || (KD == ND && !DIRECT), "scattered output reuses the input rows' lane mapping");
    extern __shared__ __align__(16) float smem[];
    float* Ws = smem;                                       // [KD][ND]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float* Xw = smem + KD * ND + wave * 32 * XS;            // [32][XS] private to this wavefront
    const int m = lane & 31, kh = lane >> 5;
    const int ci = lane % LPRI, ri = lane / LPRI, co = lane % LPRO, ro = lane / LPRO;
    const int t0 = t.chunk_tile[chunk], t1 = t.chunk_tile[chunk + 1];
    for (int ta = t0; ta < t1;) {
        const int tb = run_end(t.tile_seg, ta, t1, lane);
        const int seg = t.tile_seg[ta];
        const int ra = t.tile_row0[ta], rbnd = t.tile_row1[tb - 1];   // rows [ra, rbnd) of this segment
        const int nu = (rbnd - ra + 31) / 32;
        __syncthreads();                                    // every wavefront is done with the previous weight
        const float4* Wg = reinterpret_cast<const float4*>(W + (size_t)seg * KD * ND);
        for (int i = tid; i < KD * ND / 4; i += 64 * NW) reinterpret_cast<float4*>(Ws)[i] = Wg[i];
        __syncthreads();
        float4 wv = make_float4(0.f, 0.f, 0.f, 0.f);
        if (VEC) wv = *reinterpret_cast<const float4*>(vec + (size_t)seg * ND + co * 4);
        // lanes per head of an output row (a power of two, like the head count), and its log2
        const int lls = (31 - __clz(LPRO)) - (VEC ? 31 - __clz(s_heads) : 0), lph = 1 << lls;
        // Rows past the end of the run are clamped to its last row, so every load below is
        // unconditional; what they bring in is never stored.  LANEIDX: lane r keeps the index of row r (one register for NX)
        // and hands it to the lanes that load the row.
        constexpr bool LANEIDX = GATHER && KD == 128;
        v4f xr[NX];
        int gi[LANEIDX ? 1 : NX], gcur[SCATTER ? NX : 1];
        int ti = 0, tcur = 0;                               // XSEL: to[] of row (lane & 31), like gi and gcur
#define RGNN_FETCH_IDX(U)                                                           \
    if (XSEL) ti = to[min(ra + (U) * 32 + m, rbnd - 1)];                            \
    if (LANEIDX) gi[0] = gather[min(ra + (U) * 32 + m, rbnd - 1)];                  \
    else {                                                                          \
        _Pragma("unroll") for (int it = 0; it < NX; ++it) {                         \
            const int row_ = min(ra + (U) * 32 + ri + it * RPI, rbnd - 1);          \
            gi[LANEIDX ? 0 : it] = GATHER ? gather[row_] : row_;                    \
        }                                                                           \
    }
#define RGNN_FETCH_ROWS()                                                           \
    _Pragma("unroll") for (int it = 0; it < NX; ++it) {                             \
        const int g_ = LANEIDX ? __shfl(gi[0], ri + it * RPI) : gi[LANEIDX ? 0 : it]; \
        xr[it] = *reinterpret_cast<const v4f*>(input_row<KD, XSEL>(X, X2, g_) + ci * 4); \
        if (SCATTER) gcur[SCATTER ? it : 0] = g_;                                   \
    }                                                                               \
    if (XSEL) tcur = ti;
        RGNN_FETCH_IDX(wave)
        RGNN_FETCH_ROWS()
        RGNN_FETCH_IDX(wave + NW)
        for (int u = wave; u < nu; u += NW) {
            int gout[SCATTER ? NX : 1];
            const int tout = tcur;
            if (SCATTER) {
#pragma unroll
                for (int it = 0; it < NX; ++it) gout[SCATTER ? it : 0] = gcur[SCATTER ? it : 0];
            }
            v16f acc[CB];
#pragma unroll
            for (int b = 0; b < CB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
            // (ACCUM: the rows of Y are asked for before the next unit's rows, or the wait for them would drain those: 21.4 us
            // became 18.4 at 120k rows of width 64)
            // (the lane's place is made opaque so that the rows' addresses are formed here, not kept across the loop)
            int at = 4 * kh * (OS * ND) + m;
            asm volatile("" : "+v"(at));
            const int left = rbnd - (ra + u * 32);
            const bool full = left >= 32;
            float* const yu = Y + (size_t)(ra + u * 32) * (OS * ND) + at;   // DIRECT: this lane's first row and column
            float old1[ACCUM && DIRECT ? CB * 16 : 1];
            v4f old[ACCUM && !DIRECT ? NO : 1];
            if (ACCUM && DIRECT) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
#pragma unroll
                    for (int b = 0; b < CB; ++b)
                        old1[DIRECT && ACCUM ? b * 16 + v : 0] = yu[(full ? acc_row(v, 0) : min(acc_row(v, kh), left - 1) - 4 * kh) * (OS * ND) + b * 32];
            } else if (ACCUM) {
#pragma unroll
                for (int it = 0; it < NO; ++it)
                    old[ACCUM && !DIRECT ? it : 0] = *reinterpret_cast<const v4f*>(Y + (size_t)min(ra + u * 32 + ro + it * RPO, rbnd - 1) * (OS * ND) + co * 4);
            }
#pragma unroll
            for (int ph = 0; ph < PH; ++ph) {
                // columns [ph, ph + 1) * KS / 2 of both halves of k: 4 * ci = kh' * KD / 2 + ph * KS / 2 + column
                if (PH == 1 || ((ci >> 3) & 1) == ph) {
                    const int c = PH == 1 ? ci * 4 : (ci >> 4) * (KS / 2) + (ci & 7) * 4;
#pragma unroll
                    for (int it = 0; it < NX; ++it) *reinterpret_cast<v4f*>(Xw + (ri + it * RPI) * XS + c) = xr[it];
                }
                wave_lds_fence();
                if (ph == PH - 1) {
                    RGNN_FETCH_ROWS()             // unit u + NW
                    RGNN_FETCH_IDX(u + 2 * NW)
                }
#pragma unroll 2
                for (int tt = 0; tt < KS / 8; ++tt) {
                    const int k0 = kh * (KD / 2) + ph * (KS / 2) + 4 * tt;
                    const float4 a4 = *reinterpret_cast<const float4*>(Xw + m * XS + kh * (KS / 2) + 4 * tt);
                    const float av[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int b = 0; b < CB; ++b) acc[b] = mfma32(av[i], Ws[(k0 + i) * ND + b * 32 + m], acc[b]);
                }
                wave_lds_fence();             // all reads of the input rows are done before the stage is overwritten
            }
            if (DIRECT) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (full || acc_row(v, kh) < left) {
                        float* const yx = Y + (size_t)(XSEL ? row_of_half(tout, acc_row(v, 0), kh) : 0) * (OS * ND) + m;
#pragma unroll
                        for (int b = 0; b < CB; ++b) {
                            float y = acc[b][v];
                            if (ACCUM) {
                                y += old1[DIRECT && ACCUM ? b * 16 + v : 0];
                                if (relu) y = y > 0.f ? y : 0.f;
                            }
                            __builtin_nontemporal_store(y, XSEL ? yx + b * 32 : yu + acc_row(v, 0) * (OS * ND) + b * 32);
                        }
                    }
            } else {
#pragma unroll
                for (int b = 0; b < CB; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) Xw[acc_row(v, kh) * XS + b * 32 + m] = acc[b][v];
                wave_lds_fence();
#pragma unroll
                for (int it = 0; it < NO; ++it) {
                    const int r = ro + it * RPO, row = ra + u * 32 + r;
                    const bool ok = row < rbnd;
                    float4 y = *reinterpret_cast<const float4*>(Xw + r * XS + co * 4);
                    const size_t d = XSEL ? (size_t)__shfl(tout, r) : SCATTER ? (size_t)gout[SCATTER ? it : 0] : (size_t)min(row, rbnd - 1);
                    float4* yp = reinterpret_cast<float4*>(Y + d * (OS * ND) + co * 4);
                    if (ACCUM) {
                        const v4f o = old[ACCUM && !DIRECT ? it : 0];
                        y.x += o[0]; y.y += o[1]; y.z += o[2]; y.w += o[3];
                        if (relu) y = positive(y);
                    }
                    if (ok) {   // rows of a large tensor that is read again only after it has left the caches: non-temporal
                        const v4f yv = {y.x, y.y, y.z, y.w};
                        __builtin_nontemporal_store(yv, reinterpret_cast<v4f*>(yp));
                    }
                    if (VEC) {
                        // the lanes of a head's column slice are added (the slices are aligned groups of lph lanes)
                        float sdot = y.x * wv.x + y.y * wv.y + y.z * wv.z + y.w * wv.w;
#pragma unroll
                        for (int o = LPRO / 2; o > 0; o >>= 1) {
                            const float other = __shfl_xor(sdot, o);
                            if (o < lph) sdot += other;
                        }
                        if (ok && (co & (lph - 1)) == 0) s_out[(size_t)row * s_heads + (co >> lls)] = sdot;
                    }
                }
                wave_lds_fence();         // the stage is read out before the next unit's rows overwrite it
            }
        }
#undef RGNN_FETCH_IDX
#undef RGNN_FETCH_ROWS
        ta = tb;
    }
}

template <int KD, int ND, bool GATHER, bool SCATTER, bool ACCUM, bool VEC, bool FOLD = false, bool XSEL = false>
__global__ __launch_bounds__((64 * FwdShape<KD, ND, VEC, ACCUM>::NW))
void typed_linear_fwd_wave_kernel(TileArgs t, const float* __restrict__ X, const int32_t* __restrict__ gather,
                                  const float* __restrict__ W, float* __restrict__ Y, const float* __restrict__ vec,
                                  float* __restrict__ s_out, int s_heads, int relu, FoldArgs fold, const float* __restrict__ X2,
                                  const int32_t* __restrict__ to) {
    // RGAT: the folded vectors that the kernel after this one reads (a launch of their own cost 5 us behind this one)
    if (FOLD && (int)blockIdx.x >= (int)gridDim.x - fold.blocks) {
        if (threadIdx.x < 256) fold_weight_block(fold, blockIdx.x - (gridDim.x - fold.blocks));
        return;
    }
    fwd_wave<KD, ND, GATHER, SCATTER, ACCUM, VEC, 1, XSEL>(t, blockIdx.x, X, gather, W, Y, vec, s_out, s_heads, relu, X2, to);
}

// Several products that do not depend on each other in one launch (HGT: a node linear, rows gathered and scattered, and the two
// linears of the pairs, whose results lie side by side): workgroup b takes the b-th chunk of the jobs' chunks in a row.  Short
// products leave the chip half empty at their ends, and each costs a launch: 30k nodes and 75k pairs of width 64, 12.4 + 21.9 + 17.7
// us one by one, 29 together.
struct FwdJob { TileArgs t; int chunks, pairs; const float* X; const int32_t* gather; const float* W; float* Y; };
struct BwdJob {
    TileArgs t; int chunks, pairs; const float* X; const int32_t* gather; const float* W; const float* dY; float* dX; float* part;
};
constexpr int kMaxJobs = 3;
struct FwdJobs { FwdJob job[kMaxJobs]; int n; };
struct BwdJobs { BwdJob job[kMaxJobs]; int n; };
template <typename J>
__device__ __forceinline__ int job_of(const J& jobs, int& chunk) {
    int k = 0;
    while (k + 1 < jobs.n && chunk >= jobs.job[k].chunks) chunk -= jobs.job[k++].chunks;
    return k;
}
template <int D>
__global__ __launch_bounds__((64 * FwdShape<D, D, false, false>::NW)) void typed_linear_fwd_jobs_kernel(FwdJobs jobs) {
    int chunk = blockIdx.x;
    const FwdJob& j = jobs.job[job_of(jobs, chunk)];
    if (j.pairs) fwd_wave<D, D, true, false, false, false, 2>(j.t, chunk, j.X, j.gather, j.W, j.Y, nullptr, nullptr, 1, 0);
    else fwd_wave<D, D, true, true, false, false, 1>(j.t, chunk, j.X, j.gather, j.W, j.Y, nullptr, nullptr, 1, 0);
}

// Backward of a segment's rows:
//   dXrow[i]  = dY[i] W^T + rowscale[i] * xvec[seg]   (MFMA, contraction over the output features;
//                                                     the rank-1 term is added when the row is stored)
//   dW[seg]   = sum_i X[g(i)]^T dY[i]                 (MFMA, contraction over the rows)
//   Avec[seg] = sum_i rowscale[i] X[g(i)]             (vector ALU)
// With dY_eff = dY + rowscale (x) v, xvec = W v gives dXrow = dY_eff W^T exactly, and the caller
// completes dW = X^T dY_eff by adding Avec^T (x) v; dY_eff itself is never formed.
//
// Backward, wave-independent: eight wavefronts per workgroup, each owning 32-row units of
// the run.  Per unit a wavefront forms dXrow = dY W^T (+ rowscale (x) xvec) and adds its
// rows' contribution, summed over the unit first, to the full KD x ND weight gradient (KB*NB blocks, kept in
// registers for the whole run) and to Avec.  At the end of a run the eight wavefronts' partial weight
// gradients are summed through LDS and written to the chunk's slot.
//
// SEL (row selector): row i of dY is either dY[ysel[i]] or, when the top bit of ysel[i] is set, row
// ysel[i] & 0x7FFFFFFF of a second tensor times a per-row scale; rowscale[i] and that scale come as one
// (rowscale, scale) pair per row.  (RGAT: the gradient row of a (source,
// relation) pair with a single edge is att_e * dOut[dst_e]; it is read from dOut here instead of
// being written out per pair first.)  A lane keeps the selector and the scale of one row of the unit
// and hands them to the lanes that load or store that row with a cross-lane read.
//
// HS > 0 (row selector with HS heads, instead of RS): the columns form HS equal slices; a selected row is
//   dY_alt[row] * a[h] + b[h] * wvec[seg]   on the columns of slice h,
// with (b[0..HS), a[0..HS)) = hcoef[i] per row i.  (Multi-head RGAT: the complete gradient row of a single-edge
// pair, att_e^h dOut[dst_e] + dz_e^h w_s[r] per head, is formed while the row is staged; rows that are not
// selected come from dY as they are.)  The slot's vector part then holds HS vectors, sum over the rows of
// b[h] * X[g(i)] for h < HS (selected or not: b is the row's rowscale per head).
//
// SEL without RS or HS (RGCN): the same with the scale alone, from `scale` (null: 1).  The gradient rows of the single-edge
// pairs (74 % of the pairs of 1.2M edges) are then neither written by the pair-major walk nor read from where it put them,
// and are read from dOut, a table small enough for the caches: 832k pairs, 32 -> 64 columns, walk 79 -> 30 us, this kernel
// 87 -> 92 us; 2.15M pairs of width 64, walk 226 -> 90 us, this kernel 345 -> 373 us.
//
// XSEL (rows per run): input rows from two tensors as in the forward, X or x2, and row i of dY is dY[sel[i]].  2: the input row counts
// scale[n] times, n = num[i] (RGAT: the weight of the run), and dot[n] = dXrow[i] . (scale[n] input row i).
struct RowSelect {
    const int32_t* sel; const float* alt; const float2* ds_scale; const float* scale; const float* hcoef; const float* wvec; const float* x2;
    float* dot; const int32_t* num;
};
// DS: the rows of dY are DS * ND floats apart (not with SEL).
template <int KD, int ND, bool GATHER, bool DYG, bool SCATTER, bool RS, bool SEL = false, int HS = 0, int DS = 1, int XSEL = 0>
__device__ __forceinline__ void bwd_wave(const TileArgs& t, int chunk, const float* __restrict__ X, const int32_t* __restrict__ gather,
                                         const float* __restrict__ W, const float* __restrict__ dY, float* __restrict__ dXrow,
                                         const float* __restrict__ rowscale, const float* __restrict__ vec,
                                         float* __restrict__ part, const RowSelect& ys) {
    static_assert(!SEL || (!DYG && DS == 1), "the row selector replaces the dY gather");
    static_assert(HS == 0 || (SEL && !RS && (HS == 2 || HS == 4)), "per-head row selector: two or four heads, no rowscale");
    static_assert(!XSEL || (GATHER && !SCATTER && SEL && !RS && HS == 0), "two input tensors: gathered rows, dY through its own list");
    constexpr int NW = 8;
    constexpr int XS = KD + 4, YS = (ND > KD ? ND : KD) + 4, WS = ND + 1;
    constexpr int KB = KD / 32, NB = ND / 32, WB = KB * NB;
    constexpr int NA = HS ? HS : 1;                         // vectors in a slot's vector part
    constexpr int SLOT = KD * ND + NA * KD;
    constexpr int LPRX = KD / 4, RPX = 64 / LPRX, NXR = 32 / RPX;
    constexpr int LPRY = ND / 4, RPY = 64 / LPRY, NYR = 32 / RPY;
    constexpr int WREG = 32 * XS + 32 * YS + 32;            // floats of LDS per wavefront
    static_assert(!(DYG || SCATTER) || KD == ND, "gathered dY / scattered dXrow reuse the X rows' lane mapping");
    extern __shared__ __align__(16) float smem[];
    float* Ws = smem;                                       // [KD][WS]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float* Xw = smem + KD * WS + wave * WREG;               // [32][XS]  gathered input rows
    float* Yw = Xw + 32 * XS;                               // [32][YS]  dY rows, then the dXrow stage
    float* dsw = Yw + 32 * YS;                              // [32]      rowscale of the unit's rows
    const int m = lane & 31, kh = lane >> 5;
    const int cx = lane % LPRX, rx = lane / LPRX, cy = lane % LPRY, ry = lane / LPRY;
    const int t0 = t.chunk_tile[chunk], t1 = t.chunk_tile[chunk + 1];
    int slot = t.chunk_slot[chunk];
    for (int ta = t0; ta < t1; ++slot) {
        const int tb = run_end(t.tile_seg, ta, t1, lane);
        const int seg = t.tile_seg[ta];
        const int ra = t.tile_row0[ta], rbnd = t.tile_row1[tb - 1];
        const int nu = (rbnd - ra + 31) / 32;
        __syncthreads();                                    // previous run's flush has read the LDS regions
        {
            const float* Wg = W + (size_t)seg * KD * ND;
            for (int i = tid; i < KD * ND; i += 64 * NW) Ws[(i / ND) * WS + (i % ND)] = Wg[i];
        }
        __syncthreads();
        float4 xv = make_float4(0.f, 0.f, 0.f, 0.f);
        if (RS && vec) xv = *reinterpret_cast<const float4*>(vec + (size_t)seg * KD + cx * 4);
        if (HS) xv = *reinterpret_cast<const float4*>(ys.wvec + (size_t)seg * ND + cy * 4);   // this lane's columns of wvec[seg]
        v16f accw[WB];
#pragma unroll
        for (int b = 0; b < WB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) accw[b][v] = 0.f;
        float pa[KB];                                       // partial of Avec[kb * 32 + m] over the rows of parity kh
        v4f pah[HS ? KB : 1];                               // HS: the same for heads 0..3 (element h)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            pa[kb] = 0.f;
            pah[HS ? kb : 0] = v4f{0.f, 0.f, 0.f, 0.f};
        }
        // Rows past the end of the run are clamped to its last row (loads stay unconditional)
        // and zeroed when they are written to LDS, so they add nothing to the weight gradient.
        v4f xr[NXR], yr[NYR];
        float dsr = 0.f;
        int gi[NXR], gcur[NXR];
        int nmn = 0, nmc = 0; // XSEL 2: num of row (lane & 31) of the unit whose rows are fetched next, and of the one in yr
        int ysn = 0;          // SEL: selector of row (lane & 31) of the unit whose rows are fetched next
        float alr = 1.f;      // SEL: scale of row (lane & 31) of the unit whose rows are in yr
        // HS: (b[h0], b[h0 + 1], a[h0], a[h0 + 1]) of row (lane & 31) of the unit whose rows are in yr, a = 1 for a row
        // that is not selected (hon false); with four heads the upper half of the wavefront keeps heads 2 and 3 (h0 = 2)
        float hcf[4] = {0.f, 0.f, 1.f, 1.f};
        bool hon = false;
        const int h0 = HS == 4 ? 2 * (lane >> 5) : 0;
        // LANEIDX: the gather index of row (lane & 31) is kept by that lane and handed to the lanes that
        // load the row with a cross-lane read (one register instead of NXR); the variants that reuse the
        // indices for dY or for the scattered store keep them per load.
        constexpr bool LANEIDX = GATHER && !DYG && !SCATTER;
        int gsn = 0;
        auto fetch_idx = [&](int u) {
            if (LANEIDX) {
                gsn = gather[min(ra + u * 32 + (lane & 31), rbnd - 1)];
            } else {
#pragma unroll
                for (int it = 0; it < NXR; ++it) {
                    const int row = min(ra + u * 32 + rx + it * RPX, rbnd - 1);
                    gi[it] = GATHER ? gather[row] : row;
                }
            }
            if (SEL) ysn = ys.sel[min(ra + u * 32 + (lane & 31), rbnd - 1)];
            if (XSEL == 2) nmn = ys.num[min(ra + u * 32 + (lane & 31), rbnd - 1)];
        };
        auto fetch = [&](int u) {
#pragma unroll
            for (int it = 0; it < NXR; ++it) {
                const int gx = LANEIDX ? __shfl(gsn, rx + it * RPX) : gi[it];
                xr[it] = *reinterpret_cast<const v4f*>(input_row<KD, (XSEL > 0)>(X, ys.x2, gx) + cx * 4);
                gcur[it] = gx;
            }
#pragma unroll
            for (int it = 0; it < NYR; ++it) {
                if (XSEL) {
                    yr[it] = *reinterpret_cast<const v4f*>(dY + (size_t)__shfl(ysn, ry + it * RPY) * ND + cy * 4);
                } else if (SEL) {
                    const int sl = __shfl(ysn, ry + it * RPY);
                    const float* base = sl < 0 ? ys.alt : dY;
                    yr[it] = *reinterpret_cast<const v4f*>(base + (size_t)(sl & 0x7FFFFFFF) * ND + cy * 4);
                } else {
                    const size_t s2 = DYG ? (size_t)gi[it] : (size_t)min(ra + u * 32 + ry + it * RPY, rbnd - 1);
                    yr[it] = *reinterpret_cast<const v4f*>(dY + s2 * (DS * ND) + cy * 4);
                }
            }
            if (HS) {
                const float* hp = ys.hcoef + (size_t)min(ra + u * 32 + (lane & 31), rbnd - 1) * 2 * HS + h0;
                const float2 bb = *reinterpret_cast<const float2*>(hp), aa = *reinterpret_cast<const float2*>(hp + HS);
                hon = ysn < 0;
                hcf[0] = bb.x; hcf[1] = bb.y;
                hcf[2] = hon ? aa.x : 1.f; hcf[3] = hon ? aa.y : 1.f;
            } else if (SEL && RS) {
                const float2 pr = ys.ds_scale[min(ra + u * 32 + (lane & 31), rbnd - 1)];
                dsr = pr.x;
                alr = ysn < 0 ? pr.y : 1.f;
            } else if (XSEL == 2) {
                nmc = nmn;
                alr = ys.scale[nmn];
            } else if (SEL && !XSEL) {
                // without scales the load goes to the selectors (any bits) and is not used: no conditional load
                const float* from = ys.scale ? ys.scale : reinterpret_cast<const float*>(ys.sel);
                const float sc = from[min(ra + u * 32 + (lane & 31), rbnd - 1)];
                alr = ys.scale && ysn < 0 ? sc : 1.f;
            } else if (RS) {
                dsr = rowscale[min(ra + u * 32 + (lane & 31), rbnd - 1)];
            }
        };
        fetch_idx(wave);
        fetch(wave);
        fetch_idx(wave + NW);
        for (int u = wave; u < nu; u += NW) {
            const int rows_left = rbnd - (ra + u * 32);      // rows of this unit that exist (may exceed 32)
            const int num = nmc;
            int gout[NXR];
#pragma unroll
            for (int it = 0; it < NXR; ++it) {
                const bool ok = rx + it * RPX < rows_left;
                v4f v = xr[it];
                if (XSEL == 2) {
                    const float sc = __shfl(alr, rx + it * RPX);
                    v = v4f{v[0] * sc, v[1] * sc, v[2] * sc, v[3] * sc};
                }
                if (!ok) v = v4f{0.f, 0.f, 0.f, 0.f};
                *reinterpret_cast<v4f*>(Xw + (rx + it * RPX) * XS + cx * 4) = v;
                gout[it] = gcur[it];
            }
#pragma unroll
            for (int it = 0; it < NYR; ++it) {
                const bool ok = ry + it * RPY < rows_left;
                v4f v = yr[it];
                if (HS) {
                    // coefficients of this lane's head from the lane that keeps them for the row
                    const int hd = cy / (LPRY / (HS ? HS : 1));
                    const int from = ry + it * RPY + (HS == 4 ? 32 * (hd >> 1) : 0);
                    const float b0 = __shfl(hon ? hcf[0] : 0.f, from), b1 = __shfl(hon ? hcf[1] : 0.f, from);
                    const float a0 = __shfl(hcf[2], from), a1 = __shfl(hcf[3], from);
                    const float bq = hd & 1 ? b1 : b0, aq = hd & 1 ? a1 : a0;
                    v = v4f{v[0] * aq + bq * xv.x, v[1] * aq + bq * xv.y, v[2] * aq + bq * xv.z, v[3] * aq + bq * xv.w};
                } else if (SEL && !XSEL) {
                    const float sc = __shfl(alr, ry + it * RPY);
                    v = v4f{v[0] * sc, v[1] * sc, v[2] * sc, v[3] * sc};
                }
                if (!ok) v = v4f{0.f, 0.f, 0.f, 0.f};
                *reinterpret_cast<v4f*>(Yw + (ry + it * RPY) * YS + cy * 4) = v;
            }
            const float dsc = RS && (lane & 31) < rows_left ? dsr : 0.f;   // rowscale of row (lane & 31), zero past the end
            if (RS && lane < 32) dsw[lane] = dsc;
            if (HS) {
                // the row's rowscale per head goes into the four spare floats that end its row of Xw (zero past the end);
                // the weight-gradient section reads them back row by row
                static_assert(XS - KD == 4, "the spare floats of an X row hold the per-head rowscale");
                const bool ok = (lane & 31) < rows_left;
                if (HS == 4 || lane < 32)
                    *reinterpret_cast<float2*>(Xw + (lane & 31) * XS + KD + h0) = make_float2(ok ? hcf[0] : 0.f, ok ? hcf[1] : 0.f);
            }
            wave_lds_fence();
            fetch(u + NW);
            fetch_idx(u + 2 * NW);
            // The wavefront that is in its MFMA section goes first at instruction issue: the other wavefront
            // of the SIMD then fills the gaps with its loads and stores instead of interleaving its own MFMAs.
            __builtin_amdgcn_s_setprio(2);
            // Weight gradient: KD x ND, contraction over the unit's 32 rows (two rows per MFMA), one 32 x 32 block at a
            // time.  A unit's products are summed on their own and then added to the running gradient: one rounding at
            // the gradient's magnitude per 32 rows instead of sixteen.  With a whole chunk in one chain of MFMAs the
            // error of dW against 64 bits grows with the chunk's length (7.3M pairs in 256 chunks: 9.1e-7; so: 2.7e-7).
            // This section comes before the dXrow one, whose accumulators have to live until the rows are stored: the
            // other way round the unit's block spills.  The rows' contribution to Avec rides along with the first
            // columns: lane (m, kh) holds X[2 s + kh][kb * 32 + m] as its A operand and adds rowscale[2 s + kh] times it
            // to its partial of column kb * 32 + m.  With heads, a 4x4x1 MFMA does that for four heads at once: each
            // group of four lanes forms the outer product of the rowscale of its row for heads 0..3 (lane j of the
            // group brings head j's) with the group's four X values, and lane (m, kh) gets the four heads' partials of
            // its column.
#pragma unroll
            for (int b = 0; b < WB; ++b) {
                const int kb = b % KB, nb = b / KB;
                float av = Xw[kh * XS + kb * 32 + m], bv = Yw[kh * YS + nb * 32 + m], pu = 0.f, c1 = 0.f;
                v4f ph{0.f, 0.f, 0.f, 0.f};
                v16f t;
#pragma unroll
                for (int v = 0; v < 16; ++v) t[v] = 0.f;
                if (HS && nb == 0) c1 = Xw[kh * XS + KD + (lane & (HS - 1))];
#pragma unroll
                for (int s2 = 0; s2 < 16; ++s2) {
                    float an = 0.f, bn = 0.f, c1n = 0.f;
                    if (s2 + 1 < 16) {
                        const int r = 2 * (s2 + 1) + kh;
                        an = Xw[r * XS + kb * 32 + m];
                        bn = Yw[r * YS + nb * 32 + m];
                        if (HS && nb == 0) c1n = Xw[r * XS + KD + (lane & (HS - 1))];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if (RS && nb == 0) {
                        const float w0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, dsc), 2 * s2));
                        const float w1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, dsc), 2 * s2 + 1));
                        pu += (kh ? w1 : w0) * av;
                    }
                    if (HS && nb == 0) ph = __builtin_amdgcn_mfma_f32_4x4x1f32(c1, av, ph, 0, 0, 0);
                    t = mfma32(av, bv, t);
                    av = an;
                    bv = bn;
                    c1 = c1n;
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    accw[b][v] += t[v];
                    asm volatile("" : "+v"(accw[b][v]));    // done here, not delayed: t's registers are needed again
                }
                __builtin_amdgcn_sched_barrier(0);
                if (RS && nb == 0) pa[kb] += pu;
                if (HS && nb == 0) pah[HS ? kb : 0] += ph;
            }
            // dXrow unit: 32 x KD, contraction over the output features.  The LDS operands of both MFMA
            // sections are read ahead of the MFMAs that use them (a ring of B operands two steps deep here,
            // one step above), so a wavefront alone on its SIMD keeps the pipe fed.
            v16f accx[KB];
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) accx[b][v] = 0.f;
            {
                const float* yrow = Yw + m * YS + kh * (ND / 2);
                const float* wcol = Ws + m * WS + kh * (ND / 2);
                float bq[3][KB];
                float4 a4 = *reinterpret_cast<const float4*>(yrow), a4n = a4;
#pragma unroll
                for (int b = 0; b < KB; ++b) {
                    bq[0][b] = wcol[b * 32 * WS];
                    bq[1][b] = wcol[b * 32 * WS + 1];
                }
#pragma unroll
                for (int s2 = 0; s2 < ND / 2; ++s2) {
                    if (s2 + 2 < ND / 2) {
#pragma unroll
                        for (int b = 0; b < KB; ++b) bq[(s2 + 2) % 3][b] = wcol[b * 32 * WS + s2 + 2];
                    }
                    if (s2 % 4 == 0 && s2 + 4 < ND / 2) a4n = *reinterpret_cast<const float4*>(yrow + s2 + 4);
                    __builtin_amdgcn_sched_barrier(0);
                    const float av = s2 % 4 == 0 ? a4.x : s2 % 4 == 1 ? a4.y : s2 % 4 == 2 ? a4.z : a4.w;
#pragma unroll
                    for (int b = 0; b < KB; ++b) accx[b] = mfma32(av, bq[s2 % 3][b], accx[b]);
                    if (s2 % 4 == 3) a4 = a4n;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(0);
            wave_lds_fence();             // all reads of Yw are done before it becomes the dXrow stage
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) Yw[acc_row(v, kh) * YS + b * 32 + m] = accx[b][v];
            wave_lds_fence();
#pragma unroll
            for (int it = 0; it < NXR; ++it) {
                const int r = rx + it * RPX;
                float4 o = *reinterpret_cast<const float4*>(Yw + r * YS + cx * 4);
                if (RS) {
                    const float sc = dsw[r];
                    o.x += sc * xv.x; o.y += sc * xv.y; o.z += sc * xv.z; o.w += sc * xv.w;
                }
                const size_t d = SCATTER ? (size_t)gout[it] : (size_t)(ra + u * 32 + r);
                if (XSEL == 2) {
                    const float p = group_sum<LPRX>(dot4(*reinterpret_cast<const float4*>(Xw + r * XS + cx * 4), o));
                    const int n = __shfl(num, r);
                    if (cx == 0 && r < rows_left) ys.dot[n] = p;
                }
                if (r < rows_left) {
                    const v4f ov = {o.x, o.y, o.z, o.w};
                    __builtin_nontemporal_store(ov, reinterpret_cast<v4f*>(dXrow + d * KD + cx * 4));
                }
            }
            wave_lds_fence();
        }
        // flush: every wavefront parks its partial weight gradient in its own LDS region, then
        // all threads add the eight copies, by halves.
        __syncthreads();
        {
            float* mine = smem + KD * WS + wave * WREG;      // holds a slot's floats (checked on the host)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        mine[(kb * 32 + acc_row(v, kh)) * ND + nb * 32 + m] = accw[nb * KB + kb][v];
#pragma unroll
            for (int h = 0; h < NA; ++h) {
                float acca = 0.f;                           // Avec[h][k = lane] (lanes < KD): both row parities added
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) {
                    const float mine_p = HS ? pah[HS ? kb : 0][h & 3] : pa[kb];
                    const float both = mine_p + __shfl_xor(mine_p, 32);
                    if (kh == kb) acca = both;
                }
                if (lane < KD) mine[KD * ND + h * KD + lane] = acca;
            }
        }
        __syncthreads();
        {
            float* ps = part + (size_t)slot * SLOT;
            for (int i = tid; i < SLOT; i += 64 * NW) {
                float c[NW];
#pragma unroll
                for (int w2 = 0; w2 < NW; ++w2) c[w2] = smem[KD * WS + w2 * WREG + i];
#pragma unroll
                for (int o = 1; o < NW; o <<= 1)
#pragma unroll
                    for (int w2 = 0; w2 < NW; w2 += 2 * o) c[w2] += c[w2 + o];
                ps[i] = c[0];
            }
        }
        ta = tb;
    }
}

template <int KD, int ND, bool GATHER, bool DYG, bool SCATTER, bool RS, bool SEL = false, int HS = 0, int DS = 1, int XSEL = 0>
__global__ __launch_bounds__(512) void typed_linear_bwd_wave_kernel(TileArgs t, const float* __restrict__ X,
                                                                    const int32_t* __restrict__ gather,
                                                                    const float* __restrict__ W,
                                                                    const float* __restrict__ dY,
                                                                    float* __restrict__ dXrow,
                                                                    const float* __restrict__ rowscale,
                                                                    const float* __restrict__ vec,
                                                                    float* __restrict__ part, RowSelect ys) {
    bwd_wave<KD, ND, GATHER, DYG, SCATTER, RS, SEL, HS, DS, XSEL>(t, blockIdx.x, X, gather, W, dY, dXrow, rowscale, vec, part, ys);
}
// The backward of the products above.  A workgroup has a compute unit to itself, and a chunk costs a load of the weight and a flush
// of the gradient whatever its length, so the chunks of all jobs together are one per compute unit (sizes as above: 30 + 29 + 21.5 us
// one by one, 47 together).
template <int D>
__global__ __launch_bounds__(512) void typed_linear_bwd_jobs_kernel(BwdJobs jobs) {
    int chunk = blockIdx.x;
    const BwdJob& j = jobs.job[job_of(jobs, chunk)];
    const RowSelect none{};
    if (j.pairs) bwd_wave<D, D, true, false, false, false, false, 0, 2>(j.t, chunk, j.X, j.gather, j.W, j.dY, j.dX, nullptr, nullptr, j.part, none);
    else bwd_wave<D, D, true, true, true, false>(j.t, chunk, j.X, j.gather, j.W, j.dY, j.dX, nullptr, nullptr, j.part, none);
}

// RGCN: the pairs' product (with the row selector or without), or the runs' (XSEL), and the self-loop's, the first `chunks` workgroups and the others; chunks
// as above (833k pairs and 120k nodes, 32 -> 64 columns: 100 and 23 us, together 110).
template <int KD, int ND, bool SEL, int XSEL>
__global__ __launch_bounds__(512) void typed_linear_bwd_loop_kernel(BwdJob pair, RowSelect ys, BwdJob loop) {
    const RowSelect none{};
    if ((int)blockIdx.x < pair.chunks)
        bwd_wave<KD, ND, true, false, false, false, SEL, 0, 1, XSEL>(pair.t, blockIdx.x, pair.X, pair.gather, pair.W, pair.dY, pair.dX, nullptr, nullptr, pair.part, ys);
    else
        bwd_wave<KD, ND, false, false, false, false>(loop.t, blockIdx.x - pair.chunks, loop.X, nullptr, loop.W, loop.dY, loop.dX, nullptr, nullptr, loop.part, none);
}

// ---------------------------------------------------------------------------------------
static TileArgs tile_args(const TileList& t) {
    return TileArgs{t.tile_seg, t.tile_row0, t.tile_row1, t.chunk_tile, t.chunk_slot};
}

template <int KD, int ND, bool GATHER, bool SCATTER, bool ACCUM, bool VEC, bool FOLD = false, bool XSEL = false>
static rgnn_status_t launch_fwd_wave(const TypedLinearArgs& a, hipStream_t st) {
    using S = FwdShape<KD, ND, VEC, ACCUM>;
    constexpr size_t lds = S::LDS;
    auto kern = typed_linear_fwd_wave_kernel<KD, ND, GATHER, SCATTER, ACCUM, VEC, FOLD, XSEL>;
    RGNN_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds));
    KernelTimer kt(st, a.label ? a.label : "typed_linear_fwd");
    const FoldArgs fold = a.fold ? *a.fold : FoldArgs{};
    hipLaunchKernelGGL(kern, dim3(a.tiles->num_chunks + fold.blocks), dim3(64 * S::NW), lds, st, tile_args(*a.tiles), a.X, a.gather, a.W, a.Y,
                       a.vec, a.s_out, a.s_heads, a.relu, fold, a.X2, a.to);
    RGNN_HIP(hipGetLastError());
    return RGNN_OK;
}

template <int KD, int ND>
static rgnn_status_t launch_fwd(const TypedLinearArgs& a, hipStream_t st) {
    // the combinations the layers use
    const bool g = a.gather != nullptr, sc = g && a.scatter_out, ac = a.accumulate != 0, v = a.vec != nullptr;
    if (v && (a.s_heads < 1 || (a.s_heads & (a.s_heads - 1)) || a.s_heads > ND / 4))
        RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear: %d heads for the row-vector products at width %d", a.s_heads, ND);
    if (a.fold && (!g || sc || ac || v || a.fold->nd % 32)) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear forward: folds go with plain products of gathered rows");
    if (a.relu && !ac) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear forward: the activation is built into the accumulating variant only");
    if (a.y_stride != 1) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear forward: output rows two widths apart are built in the launches of several products only");
    if (a.X2) {
        if (!g || sc || ac || v || a.fold || !a.to) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear forward: two input tensors go with plain products of gathered rows");
        return launch_fwd_wave<KD, ND, true, false, false, false, false, true>(a, st);
    }
    if (g && !sc && !ac && v) return launch_fwd_wave<KD, ND, true, false, false, true>(a, st);
    if (g && !sc && !ac && !v && a.fold) return launch_fwd_wave<KD, ND, true, false, false, false, true>(a, st);
    if (g && !sc && !ac && !v) return launch_fwd_wave<KD, ND, true, false, false, false>(a, st);
    if constexpr (KD == ND && KD < 128) {
        if (g && sc && !ac && !v) return launch_fwd_wave<KD, ND, true, true, false, false>(a, st);
    }
    if (!g && !ac && !v) return launch_fwd_wave<KD, ND, false, false, false, false>(a, st);
    if (!g && ac && !v) return launch_fwd_wave<KD, ND, false, false, true, false>(a, st);
    RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear forward: this combination of gather / scatter / accumulate / vec is not built");
}

rgnn_status_t typed_linear_fwd(int d_in, int d_out, const TypedLinearArgs& a, hipStream_t st) {
    if (a.fold && d_in == 128 && !a.sign_matters) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear forward: folds are not built into the split product");
    if (a.tiles->num_tiles == 0) return RGNN_OK;
    if (d_in == 64 && d_out == 64) return launch_fwd<64, 64>(a, st);
    if (d_in == 32 && d_out == 32) return launch_fwd<32, 32>(a, st);
    // Width 128: the split product, except where the sign of the result selects a branch of a backward (RGAT; RGCN, whose
    // activation may also be the caller's).  A value within
    // rounding of zero then decides a gradient row, and the rounding stays the one of the fp32 instructions (1.43M pairs:
    // 0.42 ms, split 0.28).
    if (d_in == 128 && d_out == 128) return a.sign_matters || a.X2 ? launch_fwd<128, 128>(a, st) : typed_linear_split_fwd(a, st);
    if (d_in == 32 && d_out == 64) return launch_fwd<32, 64>(a, st);
    if (d_in == 64 && d_out == 32) return launch_fwd<64, 32>(a, st);
    RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear: d_in = %d, d_out = %d not supported (need 32 / 64 / 128, different widths only among 32 and 64)", d_in, d_out);
}

size_t typed_linear_bwd_scratch_floats(int d_in, int d_out, const TileList& t, int vectors) {
    return (size_t)std::max(t.num_slots, 1) * ((size_t)d_in * d_out + (size_t)std::max(vectors, 1) * d_in);
}

template <int KD, int ND, bool GATHER, bool DYG, bool SCATTER, bool RS, bool SEL = false, int HS = 0, int DS = 1, int XSEL = 0>
static rgnn_status_t launch_bwd_wave(const TypedLinearBwdArgs& a, hipStream_t st) {
    constexpr int WREG = 32 * (KD + 4) + 32 * ((ND > KD ? ND : KD) + 4) + 32;
    static_assert(WREG >= KD * ND + (HS ? HS : 1) * KD, "per-wavefront LDS region must hold a weight-gradient copy");
    const size_t lds = sizeof(float) * (KD * (ND + 1) + 8 * WREG);
    auto kern = typed_linear_bwd_wave_kernel<KD, ND, GATHER, DYG, SCATTER, RS, SEL, HS, DS, XSEL>;
    RGNN_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds));
    KernelTimer kt(st, a.label ? a.label : "typed_linear_bwd");
    hipLaunchKernelGGL(kern, dim3(a.tiles->num_chunks), dim3(512), lds, st, tile_args(*a.tiles), a.X, a.gather, a.W,
                       a.dY, a.dXrow, a.rowscale, a.vec, a.part, RowSelect{a.ysel, a.dY_alt, a.ds_yscale, a.yscale, a.hcoef, a.wvec, a.X2, a.rowdot, a.num});
    RGNN_HIP(hipGetLastError());
    return RGNN_OK;
}

template <int KD, int ND>
static rgnn_status_t launch_bwd(const TypedLinearBwdArgs& a, hipStream_t st) {
    if (a.tiles->num_tiles > 0) {
        bool done = false;
        if constexpr (KD == 128 && ND == 128) {
            RGNN_TRY(typed_linear_split_bwd(a, st));
            done = true;
        }
        if constexpr (KD <= 64 && ND <= 64) {
            const bool g = a.gather != nullptr, dg = g && a.dy_gathered, sc = g && a.scatter_dx, rs = a.rowscale != nullptr;
            done = true;
            if (a.X2) {
                if (!(g && a.ysel && !dg && !sc && !rs) || a.dY_alt || a.vec || a.ds_yscale || a.hcoef || a.dy_stride != 1)
                    RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear backward: two input tensors go with gathered X, a list of the dY rows and scales at most");
                if (a.yscale && !(a.rowdot && a.num)) RGNN_FAIL(RGNN_EINVAL, "typed linear backward: scales of input rows go with numbers and products");
                if (a.yscale) RGNN_TRY((launch_bwd_wave<KD, ND, true, false, false, false, true, 0, 1, 2>(a, st)));
                else RGNN_TRY((launch_bwd_wave<KD, ND, true, false, false, false, true, 0, 1, 1>(a, st)));
            } else if (a.dy_stride == 2) {
                if (!(g && !dg && !sc && !rs && !a.ysel && KD == ND))
                    RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear backward: dY rows two widths apart are built for gathered X, ungathered dY, no rowscale and no selector only");
                if constexpr (KD == ND) RGNN_TRY((launch_bwd_wave<KD, ND, true, false, false, false, false, 0, 2>(a, st)));
            } else if (a.ysel && a.hcoef) {
                if (!(g && !dg && !sc && !rs && a.dY_alt && a.wvec) || (a.sel_heads != 2 && a.sel_heads != 4) || ND % (4 * a.sel_heads))
                    RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear backward: the per-head row selector needs gathered X, ungathered dY, no rowscale, 2 or 4 heads of a multiple of 4 columns");
                if (a.sel_heads == 2) RGNN_TRY((launch_bwd_wave<KD, ND, true, false, false, false, true, 2>(a, st)));
                else RGNN_TRY((launch_bwd_wave<KD, ND, true, false, false, false, true, 4>(a, st)));
            } else if (a.ysel && !(g && !dg && !sc && !rs && a.dY_alt && (a.ds_yscale ? a.vec && !a.yscale : !a.vec)))
                RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear backward: the row selector needs gathered X, ungathered dY, and vec with the (rowscale, scale) pairs or neither");
            else if (a.ysel && a.ds_yscale) RGNN_TRY((launch_bwd_wave<KD, ND, true, false, false, true, true>(a, st)));
            else if (a.ysel) RGNN_TRY((launch_bwd_wave<KD, ND, true, false, false, false, true>(a, st)));
            else if (g && !dg && !sc && rs) RGNN_TRY((launch_bwd_wave<KD, ND, true, false, false, true>(a, st)));
            else if (g && !dg && !sc && !rs) RGNN_TRY((launch_bwd_wave<KD, ND, true, false, false, false>(a, st)));
            else if (KD == ND && g && dg && sc && !rs) {
                if constexpr (KD == ND) RGNN_TRY((launch_bwd_wave<KD, ND, true, true, true, false>(a, st)));
            } else if (!g && !rs) RGNN_TRY((launch_bwd_wave<KD, ND, false, false, false, false>(a, st)));
            else done = false;
        }
        if (!done) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear backward: this combination of gather / scatter / rowscale is not built");
    }
    const int kd = KD * (KD <= 64 && a.ysel && a.hcoef ? a.sel_heads : 1);
    return typed_linear_slot_reduce(*a.tiles, a.part, KD * ND, kd, a.dW, a.Avec, st, a.sums);
}

rgnn_status_t typed_linear_bwd(int d_in, int d_out, const TypedLinearBwdArgs& a, hipStream_t st) {
    if (d_in == 64 && d_out == 64) return launch_bwd<64, 64>(a, st);
    if (d_in == 32 && d_out == 32) return launch_bwd<32, 32>(a, st);
    if (d_in == 128 && d_out == 128) return launch_bwd<128, 128>(a, st);
    if (d_in == 32 && d_out == 64) return launch_bwd<32, 64>(a, st);
    if (d_in == 64 && d_out == 32) return launch_bwd<64, 32>(a, st);
    RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear backward: d_in = %d, d_out = %d not supported (need 32 / 64 / 128, different widths only among 32 and 64)", d_in, d_out);
}

template <int KD, int ND>
static rgnn_status_t launch_bwd_loop(const TypedLinearBwdArgs& p, const TypedLinearBwdArgs& l, hipStream_t st) {
    constexpr size_t lds = sizeof(float) * (KD * (ND + 1) + 8 * (32 * (KD + 4) + 32 * ((ND > KD ? ND : KD) + 4) + 32));
    const BwdJob pair{tile_args(*p.tiles), p.tiles->num_chunks, 1, p.X, p.gather, p.W, p.dY, p.dXrow, p.part};
    const BwdJob loop{tile_args(*l.tiles), l.tiles->num_chunks, 0, l.X, nullptr, l.W, l.dY, l.dXrow, l.part};
    const RowSelect ys{p.ysel, p.dY_alt, nullptr, p.yscale, nullptr, nullptr, p.X2, nullptr, nullptr};
    auto kern = p.X2 ? typed_linear_bwd_loop_kernel<KD, ND, true, 1> : p.ysel ? typed_linear_bwd_loop_kernel<KD, ND, true, 0> : typed_linear_bwd_loop_kernel<KD, ND, false, 0>;
    RGNN_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds));
    KernelTimer kt(st, "typed_linear_loop_bwd");
    hipLaunchKernelGGL(kern, dim3(pair.chunks + loop.chunks), dim3(512), lds, st, pair, ys, loop);
    RGNN_HIP(hipGetLastError());
    return RGNN_OK;
}
rgnn_status_t typed_linear_bwd_loop(int d_in, int d_out, const TypedLinearBwdArgs& p, const TypedLinearBwdArgs& l, hipStream_t st) {
    const bool plain = !p.rowscale && !l.rowscale && !p.hcoef && !p.ds_yscale && p.gather && !l.gather && !p.dy_gathered && !p.scatter_dx && !l.ysel &&
                       p.dy_stride == 1 && l.dy_stride == 1 && p.sums && l.sums && !l.X2 && (p.X2 ? p.ysel && !p.dY_alt && !p.yscale : !p.ysel || p.dY_alt);
    if (!plain) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear backward with self-loop: plain products with their sums only");
    for (const TypedLinearBwdArgs* a : {&p, &l}) RGNN_TRY(typed_linear_slot_reduce(*a->tiles, a->part, d_in * d_out, d_in, a->dW, nullptr, st, a->sums));
    if (p.tiles->num_tiles + l.tiles->num_tiles == 0) return RGNN_OK;
    if (d_in == 64 && d_out == 64) return launch_bwd_loop<64, 64>(p, l, st);
    if (d_in == 32 && d_out == 32) return launch_bwd_loop<32, 32>(p, l, st);
    if (d_in == 32 && d_out == 64) return launch_bwd_loop<32, 64>(p, l, st);
    if (d_in == 64 && d_out == 32) return launch_bwd_loop<64, 32>(p, l, st);
    RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear backward with self-loop: widths %d -> %d not built", d_in, d_out);
}
// The products of several argument sets in one launch: gathered rows, either scattered back (y_stride 1) or two widths apart.
static rgnn_status_t jobs_check(bool ok, int n) {
    if (!ok || n < 1 || n > kMaxJobs) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear jobs: one to %d plain products of gathered rows, width 32 or 64", kMaxJobs);
    return RGNN_OK;
}
rgnn_status_t typed_linear_fwd_jobs(int d, const TypedLinearArgs* a, int n, const char* label, hipStream_t st) {
    FwdJobs jobs{};
    int blocks = 0;
    for (int k = 0; k < n; ++k) {
        const bool pairs = a[k].y_stride == 2;
        RGNN_TRY(jobs_check((d == 32 || d == 64) && a[k].gather && !a[k].accumulate && !a[k].vec && (pairs ? !a[k].scatter_out : a[k].scatter_out && a[k].y_stride == 1), n));
        if (a[k].tiles->num_tiles == 0) continue;
        jobs.job[jobs.n++] = FwdJob{tile_args(*a[k].tiles), a[k].tiles->num_chunks, pairs, a[k].X, a[k].gather, a[k].W, a[k].Y};
        blocks += a[k].tiles->num_chunks;
    }
    if (blocks == 0) return RGNN_OK;
    KernelTimer kt(st, label);
#define RGNN_JOBS(D_)                                                                                               \
    do {                                                                                                            \
        constexpr size_t lds = FwdShape<D_, D_, false, false>::LDS;                                                 \
        RGNN_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(typed_linear_fwd_jobs_kernel<D_>), lds));          \
        hipLaunchKernelGGL(typed_linear_fwd_jobs_kernel<D_>, dim3(blocks), dim3(64 * FwdShape<D_, D_, false, false>::NW), lds, st, jobs); \
    } while (0)
    if (d == 64) RGNN_JOBS(64);
    else RGNN_JOBS(32);
#undef RGNN_JOBS
    RGNN_HIP(hipGetLastError());
    return RGNN_OK;
}
rgnn_status_t typed_linear_bwd_jobs(int d, const TypedLinearBwdArgs* a, int n, const char* label, hipStream_t st) {
    BwdJobs jobs{};
    int blocks = 0;
    for (int k = 0; k < n; ++k) {
        const bool pairs = a[k].dy_stride == 2;
        RGNN_TRY(jobs_check((d == 32 || d == 64) && a[k].gather && !a[k].rowscale && !a[k].ysel && a[k].sums &&
                            (pairs ? !a[k].dy_gathered && !a[k].scatter_dx : a[k].dy_gathered && a[k].scatter_dx && a[k].dy_stride == 1), n));
        RGNN_TRY(typed_linear_slot_reduce(*a[k].tiles, a[k].part, d * d, d, a[k].dW, nullptr, st, a[k].sums));
        if (a[k].tiles->num_tiles == 0) continue;
        jobs.job[jobs.n++] = BwdJob{tile_args(*a[k].tiles), a[k].tiles->num_chunks, pairs, a[k].X, a[k].gather, a[k].W, a[k].dY, a[k].dXrow, a[k].part};
        blocks += a[k].tiles->num_chunks;
    }
    if (blocks == 0) return RGNN_OK;
    KernelTimer kt(st, label);
#define RGNN_JOBS(D_)                                                                                               \
    do {                                                                                                            \
        constexpr size_t lds = sizeof(float) * (D_ * (D_ + 1) + 8 * (64 * (D_ + 4) + 32));                          \
        RGNN_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(typed_linear_bwd_jobs_kernel<D_>), lds));          \
        hipLaunchKernelGGL(typed_linear_bwd_jobs_kernel<D_>, dim3(blocks), dim3(512), lds, st, jobs);               \
    } while (0)
    if (d == 64) RGNN_JOBS(64);
    else RGNN_JOBS(32);
#undef RGNN_JOBS
    RGNN_HIP(hipGetLastError());
    return RGNN_OK;
}

}  // namespace rgnn
