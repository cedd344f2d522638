// fp32 typed linear layer of width 128 on the bf16 matrix cores, without loss of fp32 accuracy.
//
// Every fp32 operand is split into three bf16 planes, x = hi + mid + lo (round to nearest even: |mid| <= 2^-9 |x|,
// |lo| <= 2^-18 |x|), and a product is the six plane products down to 2^-18: hi hi + (hi mid + mid hi) + (hi lo + mid mid +
// lo hi); what is left out is below 2^-26 of |x y|, a quarter of a rounding of the fp32 product.  Products are exact and sums
// are fp32, one rounding per 16 terms and plane product against one per 2 terms of v_mfma_f32_32x32x2_f32, so the result is
// as close to 64 bits as that of the fp32 matrix instructions, at 16 / 6 of their rate.  (The technique: G. Henry, P. Tang,
// A. Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", ARITH 2019.)
//
// The split holds for zero and for magnitudes from 2^-110, the least fp32 whose last bit, 2^-133, is a (subnormal) bf16, to
// 3.38e38, the greatest whose bf16 is finite.  A unit of rows, or a weight's band of 32 rows or columns, with an operand
// outside is multiplied with the fp32 matrix instructions, straight from global memory (a backward whose every unit goes that
// way, RGCN, 1.43M pairs: 1.75 ms for 0.63).  NaN needs no such care: its planes are NaN.  (A
// sum within 1 % of the largest float may overflow: the product of the high planes can be that much above it.)  Without the lower bound the error of dX and
// dW, 1.1e-7 and 1.7e-7 in the range, was 2.2e-6 with one operand near 2^-116 and 3.5e-5 near 2^-120; the check costs 1.3 % of an
// RGAT forward + backward on those pairs.
//
// Why: at width 128 a row costs 32 kflop per product against 1.5 KB of traffic, twice what the fp32 matrix cores do in the time
// the rows need.  (RGAT's and RGCN's forward stay on those: the sign of a result selects a branch of their backward.)
// 1.43M pairs of 60 relations: forward 0.42 -> 0.28 ms (5.2 TB/s), backward (two kernels before, dY read
// twice) 1.18 -> 0.54 ms (4.1 TB/s; without its matrix instructions and stores, which mostly run beside the loading
// wavefronts' chain of waits, splits and LDS writes, it would be 0.37).
//
// Row selector (RGAT with one head, RGCN): rows of single-edge pairs come straight from the destinations' gradient rows, as in
// typed_linear.hip.  With 77 % such pairs, 716k in all: this kernel 307 -> 321 us (before the stores moved), RGAT's edge walk 189 -> 143 us, RGCN's pair
// walk 139 -> 52 us; at 68k pairs 48 -> 50, 31 -> 26 and 14 -> 10.
//
// A workgroup takes a chunk of 64-row tiles in units of 32 rows, one workgroup per compute unit, its wavefronts specialised:
//   4 load:     rows of unit u + 1 from registers (fetched two units ahead) split into planes in LDS; forward: result rows of
//               unit u - 1 from LDS to memory, 512 bytes each
//   4 multiply: dXrow = dY W^T (forward: Y = X W); a wavefront keeps 32 rows (columns) of W as planes in 96 registers.  Backward:
//               it stores its columns of the result itself, in whole 128-byte lines (handed back through LDS to the loading
//               wavefronts, whose chain the kernel waits for, the stores made the backward 0.61 ms with the rows of every
//               pair in one tensor, 0.65 with the row selector; now 0.54 with it).  The forward, whose loading wavefronts have
//               half the rows to split, is nearer to the memory's rate, and there whole rows win: HGT's forward at 4M edges, result
//               rows 1 KB apart, 2.86 ms with stores by column band, so 2.66 (300 relations), 2.02 and 1.87 (60), at 300k edges the same
//   4 multiply (backward only): the weight gradient X^T dY, whose row contraction reads the planes through the transposing
//               LDS read ds_read_b64_tr_b16
// The planes (and the forward's result tiles) are double-buffered and one barrier per unit separates the stages, so that splitting
// and matrix products of neighbouring units overlap (with all wavefronts going through the phases together the backward took
// 0.70 ms at the sizes above, 15,400 clocks per 64 rows of which the matrix instructions are 6,100).
// A plane is [32 rows][256 bytes], piece c (16 bytes) of row r at c ^ swz(r), as in the bf16 backward.
#include "rgnn_internal.h"
#include "device_utils.h"

namespace rgnn {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int D = 128;
constexpr int UNIT = 32;                     // rows of a unit
constexpr int PLANE = UNIT * 2 * D;          // bytes of one plane of a unit
constexpr int STAGE = UNIT * 4 * D;          // bytes of a result tile (forward)
constexpr float kSplitMax = 3.38e38f;        // largest magnitude whose bf16 rounding is finite
constexpr unsigned kSplitMin = 17u << 23;    // bits of 2^-110: smallest magnitude above zero that three planes hold exactly

struct TileArgs {
    const int32_t* tile_seg;
    const int32_t* tile_row0;
    const int32_t* tile_row1;
    const int32_t* chunk_tile;
    const int32_t* chunk_slot;
};

__device__ __forceinline__ float lo_half(unsigned u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float hi_half(unsigned u) { return __uint_as_float(u & 0xFFFF0000u); }
// planes of the pair (a, b), packed
__device__ __forceinline__ void split2(float a, float b, unsigned (&p)[3]) {
    p[0] = bf16_pack2(a, b);
    const float a1 = a - lo_half(p[0]), b1 = b - hi_half(p[0]);
    p[1] = bf16_pack2(a1, b1);
    p[2] = bf16_pack2(a1 - lo_half(p[1]), b1 - hi_half(p[1]));
}
__device__ __forceinline__ v16f mfma16(bf16x8 a, bf16x8 b, v16f c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ v16f mfma32(float a, float b, v16f c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
// Rows of unit u of the tile list: [row0, row0 + rows), rows <= 0 for the second half of a short tile.
struct Unit { int row0, rows, seg; };
struct Units {
    TileTable t;
    __device__ __forceinline__ Units(const TileArgs& a, int t0, int t1) : t(a.tile_seg, a.tile_row0, a.tile_row1, t0, t1) {}
    __device__ __forceinline__ Unit get(int u) {
        const int l = t.lane_of(u >> 1), r = t.row0_at(l) + (u & 1) * UNIT;
        return Unit{r, min(t.row1_at(l) - r, UNIT), t.seg_at(l)};
    }
};

// Two products of three-plane operands, the six plane products of each in turn, so that no matrix instruction waits for the
// one before it.  ORDER: which operand's low plane comes first.
template <int ORDER>
__device__ __forceinline__ void mfma_split2(const bf16x8 (&a)[3], const bf16x8 (&b)[3], v16f& c, const bf16x8 (&a1)[3], const bf16x8 (&b1)[3], v16f& c1) {
    constexpr int p[2][6] = {{0, 2, 1, 0, 1, 0}, {2, 0, 1, 1, 0, 0}};          // the small products first
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        c = mfma16(a[p[ORDER][i]], b[p[1 - ORDER][i]], c);
        c1 = mfma16(a1[p[ORDER][i]], b1[p[1 - ORDER][i]], c1);
    }
}

// Whether any of the operands seen is one that the split does not hold for.
struct Range {
    float mx = 0.f;
    unsigned mn = 0xFFFFFFFFu;               // least 2 * bits(|x|) - 1: zero wraps round to the top
    __device__ __forceinline__ void see(float x) {
        mx = fmaxf(mx, fabsf(x));
        mn = min(mn, (__float_as_uint(x) << 1) - 1u);
    }
    __device__ __forceinline__ bool outside() const { return mx > kSplitMax || mn < 2u * kSplitMin - 1u; }
};

// The loading threads' view of a unit: 256 threads, 32 lanes per row (16 bytes each), rows lr + 8 k.
struct Loader {
    int c4, lr;
    __device__ __forceinline__ explicit Loader(int tid) : c4(tid & 31), lr(tid >> 5) {}
    // row lr + 8 k into the planes at `t` (zeros when !ok)
    __device__ __forceinline__ void put(unsigned char* t, int k, float4 x, bool ok, Range& seen) const {
        if (!ok) x = make_float4(0.f, 0.f, 0.f, 0.f);
        const int r = lr + 8 * k, at = r * 256 + (((c4 >> 1) ^ swz(r)) << 4) + (c4 & 1) * 8;
        unsigned p[3], q[3];
        split2(x.x, x.y, p);
        split2(x.z, x.w, q);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<uint2*>(t + pl * PLANE + at) = make_uint2(p[pl], q[pl]);
        seen.see(x.x); seen.see(x.y); seen.see(x.z); seen.see(x.w);
    }
};

// Rows of a result tile: [32][512 bytes], 16-byte piece p of row r at p ^ (r & 15).
__device__ __forceinline__ float4* stage_at(unsigned char* st, int row, int piece) {
    return reinterpret_cast<float4*>(st + row * 512 + ((piece ^ (row & 15)) << 4));
}

// One 32 x 32 block (rows of the unit x this wavefront's 32 columns) of rows times W: d[v] = result[row 8 (v / 4) + 4 kh +
// v % 4][column m], or TRANS result[row m][column 8 (v / 4) + 4 kh + v % 4]; planes of the rows at `t`, of W in w; slow: from
// memory, with wp[k * WK] = W's operand and the row of lane m as row_at() says (pointer and scale).
struct RowAt { const float* p; float scale; };
template <int WK, bool TRANS, typename F>
__device__ __forceinline__ v16f multiply_rows(const unsigned char* t, const bf16x8 (&w)[3][8], int m, int kh, bool slow, const float* wp, F row_at) {
    v16f d, d1;                                            // two chains of matrix instructions
#pragma unroll
    for (int v = 0; v < 16; ++v) d[v] = d1[v] = 0.f;
    if (!slow) {
        int rm = m;
        asm volatile("" : "+v"(rm));                       // (the places in LDS are formed here, not kept across the unit loop)
        const unsigned char* row = t + rm * 256;
        const int sw = (kh ^ swz(rm)) << 4;
#pragma unroll
        for (int s = 0; s < 8; s += 2) {
            bf16x8 x[2][3], ws[2][3];
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    x[j][q] = *reinterpret_cast<const bf16x8*>(row + q * PLANE + (sw ^ ((s + j) << 5)));
                    ws[j][q] = w[q][s + j];
                }
            if (TRANS) mfma_split2<0>(ws[0], x[0], d, ws[1], x[1], d1);
            else mfma_split2<1>(x[0], ws[0], d, x[1], ws[1], d1);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) d[v] += d1[v];
    } else {
        // (the order of k is free: a half of the wavefront takes k = 64 kh + 0..63, 16 of them in flight)
        const RowAt x = row_at();
#pragma unroll 1
        for (int k = 64 * kh; k < 64 * kh + 64; k += 16) {
            float wv[16], xv[16];
            load_cols(x.p + k, xv);
            if constexpr (WK == 1) load_cols(wp + k, wv);
            else {
#pragma unroll
                for (int e = 0; e < 16; ++e) wv[e] = wp[(size_t)(k + e) * WK];
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) d = TRANS ? mfma32(wv[e], xv[e] * x.scale, d) : mfma32(xv[e] * x.scale, wv[e], d);
        }
    }
    return d;
}

// The block's rows r < rows to memory: row r at out + to[r] * ld (TO) or out + r * ld, where `out` points at the lane's column,
// with s[r] * vcol added (RS).  The wavefront writes whole 128-byte lines, two rows per store.
template <bool TO, bool RS>
__device__ __forceinline__ void store_rows(const v16f& d, float* out, int rows, int kh, int ld, const int* to, const float* s, float vcol) {
    const bool full = rows == UNIT;
    int at = 4 * kh * ld;
    asm volatile("" : "+v"(at));                           // (the rows' places are formed here, not kept across the unit loop)
    float* const mine = out + at;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = 8 * q + 4 * kh;
        int t[4];
        float sv[4];
        if (TO) {
            const int4 t4 = *reinterpret_cast<const int4*>(to + r);
            t[0] = t4.x; t[1] = t4.y; t[2] = t4.z; t[3] = t4.w;
        }
        if (RS) {
            const float4 s4 = *reinterpret_cast<const float4*>(s + r);
            sv[0] = s4.x; sv[1] = s4.y; sv[2] = s4.z; sv[3] = s4.w;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float y = d[4 * q + j];
            if (RS) y += sv[j] * vcol;
            if (full || r + j < rows) __builtin_nontemporal_store(y, TO ? out + (size_t)t[j] * ld : mine + (8 * q + j) * ld);
        }
    }
}

// planes of eight values
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8& a, bf16x8& b, bf16x8& c, Range& seen) {
    rgnn_v4u pl[3];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        unsigned p[3];
        split2(x[2 * e], x[2 * e + 1], p);
        seen.see(x[2 * e]);
        seen.see(x[2 * e + 1]);
#pragma unroll
        for (int q = 0; q < 3; ++q) pl[q][e] = p[q];
    }
    a = __builtin_bit_cast(bf16x8, pl[0]);
    b = __builtin_bit_cast(bf16x8, pl[1]);
    c = __builtin_bit_cast(bf16x8, pl[2]);
}

// Out-of-range flags, one per unit in a ring of four: the loaders set unit u + 1's flag while unit u is multiplied and
// clear unit u + 2's, which nobody reads or sets then.
__device__ __forceinline__ void clear_flag(int* bad, int u, int tid) { if (tid == 0) bad[(u + 2) & 3] = 0; }

// ------------------------------------------------------------------------------------------------ forward

struct FwdArgs {
    TileArgs t;
    const float* X;
    const int32_t* gather;
    const float* W;          // [segs][D][D]
    float* Y;
    int ldy;                 // floats from one row of Y to the next
};

template <bool SCATTER>
__device__ __forceinline__ void fwd_load(const FwdArgs& a, unsigned char* lds, int* bad, int u0, int u1) {
    constexpr int DEPTH = 3;                               // units in flight per thread: 48 KB per compute unit
    const int tid = threadIdx.x & 255;
    const Loader ld(tid);
    Units units(a.t, u0 >> 1, u1 >> 1);
    unsigned char* const St = lds + 2 * 3 * PLANE;
    // Rows are asked for DEPTH units before they are used, and their indices DEPTH units before that: loads complete in issue
    // order, so an index that is needed while newer rows are under way must be older than all rows that are not needed yet.
    float4 xr[DEPTH][4];
    int gi[2 * DEPTH][4];
    auto fetch_idx = [&](int p, int u) {
        const Unit n = units.get(min(u, u1 - 1));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            gi[p][k] = a.gather[n.row0 + min(ld.lr + 8 * k, n.rows - 1)];     // (an empty second half: the tile's last row)
        }
    };
    auto fetch = [&](int p, int q) {
#pragma unroll
        for (int k = 0; k < 4; ++k) xr[p][k] = *reinterpret_cast<const float4*>(a.X + (size_t)gi[q][k] * D + ld.c4 * 4);
    };
#pragma unroll
    for (int p = 0; p < 2 * DEPTH; ++p) fetch_idx(p, u0 + p);
#pragma unroll
    for (int p = 0; p < DEPTH; ++p) fetch(p, p);
    int gout[2][4];                                        // destination rows of the units u and u - 1
#pragma unroll
    for (int k = 0; k < 4; ++k) gout[0][k] = gout[1][k] = 0;
    for (int ub = u0 - 1; ub <= u1; ub += 2 * DEPTH) {
#pragma unroll
        for (int p = 0; p < 2 * DEPTH; ++p) {
            const int u = ub + p;
            if (u > u1) break;
            __syncthreads();
            clear_flag(bad, u, tid);
            if (u - 1 >= u0) {                             // result rows of the unit before
                const Unit n = units.get(u - 1);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int r = ld.lr + 8 * k;
                    const bool ok = r < n.rows;
                    float4 y = *stage_at(St + ((u - 1) & 1) * STAGE, r, ld.c4);
                    if (ok) {
                        float* o = a.Y + (SCATTER ? (size_t)gout[1][k] : (size_t)(n.row0 + r)) * a.ldy + ld.c4 * 4;
                        const rgnn_v4f yv = {y.x, y.y, y.z, y.w};
                        __builtin_nontemporal_store(yv, reinterpret_cast<rgnn_v4f*>(o));
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                gout[1][k] = gout[0][k];
                gout[0][k] = gi[p][k];
            }
            // (every load of the loop is unconditional, past the end it repeats the last unit: were one skipped on some path,
            // the waits would have to assume it everywhere and drain the rows under way)
            {
                const Unit n = units.get(min(u + 1, u1 - 1));
                unsigned char* const t = lds + ((u + 1) & 1) * 3 * PLANE;
                Range seen;
#pragma unroll
                for (int k = 0; k < 4; ++k) ld.put(t, k, xr[p % DEPTH][k], ld.lr + 8 * k < n.rows, seen);
                if (seen.outside()) bad[(u + 1) & 3] = 1;
                fetch_idx(p, u + 1 + 2 * DEPTH);
                fetch(p % DEPTH, (p + DEPTH) % (2 * DEPTH));
            }
        }
    }
}

__device__ __forceinline__ void fwd_multiply(const FwdArgs& a, unsigned char* lds, int* bad, int u0, int u1) {
    const int lane = threadIdx.x & 63, band = threadIdx.x >> 6, m = lane & 31, kh = lane >> 5;
    unsigned char* const St = lds + 2 * 3 * PLANE;
    Units units(a.t, u0 >> 1, u1 >> 1);
    bf16x8 w[3][8];
    int cur_seg = -1;
    bool wbad = false;
    for (int u = u0 - 1; u <= u1; ++u) {
        __syncthreads();
        if (u < u0 || u >= u1) continue;
        const Unit n = units.get(u);
        const float* const wp = a.W + (size_t)n.seg * D * D + band * 32 + m;
        if (n.seg != cur_seg) {
            cur_seg = n.seg;
            Range seen;
#pragma unroll
            for (int s = 0; s < 8; ++s) {                  // lane (m, kh) keeps W[16 s + 8 kh + 0..7][band * 32 + m]
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = wp[(size_t)(16 * s + 8 * kh + e) * D];
                split8(x, w[0][s], w[1][s], w[2][s], seen);
            }
            wbad = __any(seen.outside());
        }
        if (n.rows <= 0) continue;
        const bool slow = wbad || bad[u & 3];
        const v16f d = multiply_rows<D, true>(lds + (u & 1) * 3 * PLANE, w, m, kh, slow, wp, [&] {
            return RowAt{a.X + (size_t)a.gather[n.row0 + min(m, n.rows - 1)] * D, 1.f};
        });
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *stage_at(St + (u & 1) * STAGE, m, band * 8 + 2 * q + kh) = make_float4(d[4 * q], d[4 * q + 1], d[4 * q + 2], d[4 * q + 3]);
    }
}

// X rows through the gather list; SCATTER: Y rows as well
template <bool SCATTER>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void typed_linear_split_fwd_kernel(FwdArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];   // [2][3] planes, [2] result tiles
    __shared__ int bad[4];
    const int u0 = 2 * a.t.chunk_tile[blockIdx.x], u1 = 2 * a.t.chunk_tile[blockIdx.x + 1];
    if (threadIdx.x < 4) bad[threadIdx.x] = 0;
    __syncthreads();
    if (u0 >= u1) return;
    if (threadIdx.x >= 256) fwd_load<SCATTER>(a, lds, bad, u0, u1);
    else fwd_multiply(a, lds, bad, u0, u1);
}

// ------------------------------------------------------------------------------------------------ backward

struct BwdArgs {
    TileArgs t;
    const float* X;
    const int32_t* gather;
    const float* W;
    const float* dY;
    int ldd;                 // floats from one row of dY to the next
    float* dX;
    const float* rowscale;   // RS: dXrow[i] += rowscale[i] * vec[seg], and the slot's vector part is sum rowscale[i] X[g(i)]
    const float* vec;
    float* part;             // slots of D * D + D floats
    // SEL: row i of dY is dY[ysel[i]], or, when the top bit of ysel[i] is set, row ysel[i] & 0x7FFFFFFF of dY_alt times a
    // scale: with RS that of the pair (rowscale, scale) = ds_yscale[i], otherwise yscale[i] (null: 1)
    const int32_t* ysel;
    const float* dY_alt;
    const float2* ds_yscale;
    const float* yscale;
    const float* X2;         // XSEL: list entry g < 0 is row g & 0x7FFFFFFF of X2 (SEL is then a plain list of dY rows); 2: X rows count yscale[n] times,
    float* dot;              // n = num[i], and dot[n] = dXrow[i] . yscale[n] X row
    const int32_t* num;
};
template <int XSEL>
__device__ __forceinline__ const float* input_row(const BwdArgs& a, int g) { return (XSEL && g < 0 ? a.X2 : a.X) + (size_t)(XSEL ? g & 0x7FFFFFFF : g) * D; }
__device__ __forceinline__ const float* selected_row(const BwdArgs& a, int sl) { return (sl < 0 ? a.dY_alt : a.dY) + (size_t)(sl & 0x7FFFFFFF) * D; }
template <bool RS>
__device__ __forceinline__ float selected_scale(const BwdArgs& a, int row, int sl) {
    // (without scales the load goes to the selectors, any bits, and is not used: no conditional load)
    const float sc = RS ? a.ds_yscale[row].y : (a.yscale ? a.yscale : reinterpret_cast<const float*>(a.ysel))[row];
    return sl < 0 && (RS || a.yscale) ? sc : 1.f;
}
constexpr int SLOT = D * D + D;
struct RowOf { int to[UNIT]; float s[UNIT]; };   // destinations and rowscales of a unit's rows on its way through the pipeline
constexpr int BUF = 6 * PLANE;               // planes of a unit: X, then dY
// XSEL 2: the unit's X rows in fp32 for the products with dXrow ([2][32][512 bytes] behind the planes), whose sums over each wavefront's 32
// columns the loading wavefronts add (a ring like the flags)
constexpr int XROWS = UNIT * 4 * D;
struct DotOf { float band[4][UNIT]; int num[UNIT]; };

// A value that lane half + 2 k keeps, for the 32 lanes of that half of the wavefront (no trip through LDS).
__device__ __forceinline__ int of_row(int v, int k, int half) {
    const int a = __builtin_amdgcn_readlane(v, 2 * k), b = __builtin_amdgcn_readlane(v, 2 * k + 1);
    return half ? b : a;
}
template <bool GATHER, bool BOTH, bool RS, bool SEL, int XSEL>
__device__ __forceinline__ void bwd_load(const BwdArgs& a, unsigned char* lds, float4* avb, RowOf* row_of, DotOf* dot_of, int* bad, int u0, int u1) {
    constexpr int DEPTH = 2;                               // units in flight per thread: 64 KB per compute unit
    const int tid = threadIdx.x & 255;
    const Loader ld(tid);
    Units units(a.t, u0 >> 1, u1 >> 1);
    float4 xr[DEPTH][4], yr[DEPTH][4], av = make_float4(0.f, 0.f, 0.f, 0.f);
    // Lane j of a wavefront keeps the index, selector and scales of row jrow, its row j of the eight that the wavefront loads
    // (a register instead of four), and hands them to the 32 lanes of that row.
    const int lane = tid & 63, half = lane >> 5, jrow = 2 * (tid >> 6) + (lane & 1) + 8 * ((lane >> 1) & 3);
    int gi[2 * DEPTH], yi[2 * DEPTH];                      // indices run further ahead (see the forward)
    int ni[XSEL == 2 ? 2 * DEPTH : 1];                     // XSEL 2: num
    float rs[DEPTH], sc[DEPTH];
    auto fetch_idx = [&](int p, int u) {
        const Unit n = units.get(min(u, u1 - 1));
        const int row = n.row0 + min(jrow, n.rows - 1);    // (an empty second half: the tile's last row)
        gi[p] = GATHER ? a.gather[row] : row;
        yi[p] = SEL ? a.ysel[row] : row;
        if (XSEL == 2) ni[XSEL == 2 ? p : 0] = a.num[row];
    };
    auto fetch = [&](int p, int q, int u) {
        const Unit n = units.get(min(u, u1 - 1));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int row = n.row0 + min(ld.lr + 8 * k, n.rows - 1), g = GATHER ? of_row(gi[q], k, half) : row;
            xr[p][k] = *reinterpret_cast<const float4*>(input_row<XSEL>(a, g) + ld.c4 * 4);
            const float* const y = SEL ? selected_row(a, of_row(yi[q], k, half)) : a.dY + (size_t)(BOTH ? g : row) * a.ldd;
            yr[p][k] = *reinterpret_cast<const float4*>(y + ld.c4 * 4);
        }
        const int row = n.row0 + min(jrow, n.rows - 1);
        rs[p] = RS ? (SEL ? a.ds_yscale[row].x : a.rowscale[row]) : 0.f;
        sc[p] = XSEL == 2 ? a.yscale[ni[XSEL == 2 ? q : 0]] : SEL && !XSEL ? selected_scale<RS>(a, row, yi[q]) : 1.f;
    };
#pragma unroll
    for (int p = 0; p < 2 * DEPTH; ++p) fetch_idx(p, u0 + p);
#pragma unroll
    for (int p = 0; p < DEPTH; ++p) fetch(p, p, u0 + p);
    // the vector part of a slot: the eight threads of a column group leave their sums in avb when the segment ends, and after
    // the next barrier one of them adds them in order
    int seg = -1, slot = a.t.chunk_slot[blockIdx.x] - 1, pending = -1, pending_buf = 0;
    auto step = [&](int p, int u) __attribute__((always_inline)) {
        __syncthreads();
        clear_flag(bad, u, tid);
        if (pending >= 0 && tid < 32) {
            float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
            if (RS) {
                s = avb[pending_buf * 256 + tid];
                for (int r = 1; r < 8; ++r) fma4(s, 1.f, avb[pending_buf * 256 + r * 32 + tid]);
            }
            reinterpret_cast<float4*>(a.part + (size_t)pending * SLOT + D * D)[tid] = s;
        }
        pending = -1;
        if (XSEL == 2 && u - 1 >= u0 && tid < UNIT) {          // the rows of the unit that was multiplied before this barrier
            const Unit p = units.get(u - 1);
            DotOf& q = dot_of[(u - 1) & 3];
            if (tid < p.rows) a.dot[q.num[tid]] = (q.band[0][tid] + q.band[1][tid]) + (q.band[2][tid] + q.band[3][tid]);
        }
        const Unit n = units.get(min(u + 1, u1 - 1));
        const int next_seg = u + 1 < u1 ? n.seg : -2;
        if (next_seg != seg && u + 1 <= u1) {
            if (seg >= 0) {
                pending = slot;
                pending_buf = u & 1;
                if (RS) avb[pending_buf * 256 + tid] = av;
                av = make_float4(0.f, 0.f, 0.f, 0.f);
            }
            ++slot;
            seg = next_seg;
        }
        {                                              // (unconditional loads: see the forward)
            unsigned char* const t = lds + ((u + 1) & 1) * BUF;
            Range seen;
            float4 au = make_float4(0.f, 0.f, 0.f, 0.f);     // the unit's share first: fewer roundings at the sum's magnitude
            if (RS && lane < 8) row_of[(u + 1) & 3].s[jrow] = rs[p % DEPTH];
            if (BOTH && lane < 8) row_of[(u + 1) & 3].to[jrow] = gi[p];
            if (XSEL == 2 && lane < 8) dot_of[(u + 1) & 3].num[jrow] = ni[XSEL == 2 ? p : 0];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool ok = u + 1 < u1 && ld.lr + 8 * k < n.rows;
                float4 x = xr[p % DEPTH][k];
                if (!ok) x = make_float4(0.f, 0.f, 0.f, 0.f);
                if (XSEL == 2) {
                    const float s = __int_as_float(of_row(__float_as_int(sc[p % DEPTH]), k, half));
                    x = make_float4(x.x * s, x.y * s, x.z * s, x.w * s);
                    *reinterpret_cast<float4*>(lds + 2 * BUF + ((u + 1) & 1) * XROWS + (ld.lr + 8 * k) * 512 + ld.c4 * 16) = x;
                }
                if (RS) {
                    const float r = __int_as_float(of_row(__float_as_int(rs[p % DEPTH]), k, half));
                    fma4(au, ok ? r : 0.f, x);
                }
                ld.put(t, k, x, ok, seen);
                float4 y = yr[p % DEPTH][k];
                if (SEL && !XSEL) {
                    const float s = __int_as_float(of_row(__float_as_int(sc[p % DEPTH]), k, half));
                    y = make_float4(y.x * s, y.y * s, y.z * s, y.w * s);
                }
                ld.put(t + 3 * PLANE, k, y, ok, seen);
            }
            if (RS) fma4(av, 1.f, au);
            if (seen.outside()) bad[(u + 1) & 3] = 1;
            fetch_idx(p, u + 1 + 2 * DEPTH);
            fetch(p % DEPTH, (p + DEPTH) % (2 * DEPTH), u + 1 + DEPTH);
        }
    };
    // (whole rounds of the ring without an exit inside: a path from the middle of a round to its beginning would make the
    // waits there drain the rows under way)
    int u = u0 - 1;
    for (; u + 2 * DEPTH - 1 <= u1; u += 2 * DEPTH) {
#pragma unroll
        for (int p = 0; p < 2 * DEPTH; ++p) step(p, u + p);
    }
#pragma unroll
    for (int p = 0; p < 2 * DEPTH - 1; ++p)
        if (u + p <= u1) step(p, u + p);
}

template <bool GATHER, bool BOTH, bool RS, bool SEL, int XSEL>
__device__ __forceinline__ void bwd_multiply(const BwdArgs& a, unsigned char* lds, const RowOf* row_of, DotOf* dot_of, int* bad, int u0, int u1) {
    const int lane = threadIdx.x & 63, band = threadIdx.x >> 6, m = lane & 31, kh = lane >> 5;
    float vcol = 0.f;                                      // RS: this lane's column of vec[seg]
    Units units(a.t, u0 >> 1, u1 >> 1);
    bf16x8 w[3][8];
    int cur_seg = -1;
    bool wbad = false;
    for (int u = u0 - 1; u <= u1; ++u) {
        __syncthreads();
        if (u < u0 || u >= u1) continue;
        const Unit n = units.get(u);
        const float* const wp = a.W + (size_t)n.seg * D * D + (size_t)(band * 32 + m) * D;
        if (n.seg != cur_seg) {
            cur_seg = n.seg;
            Range seen;
#pragma unroll
            for (int s = 0; s < 8; ++s) {                  // lane (m, kh) keeps W[band * 32 + m][16 s + 8 kh + 0..7]
                float x[8];
                load_cols(wp + 16 * s + 8 * kh, x);
                split8(x, w[0][s], w[1][s], w[2][s], seen);
            }
            wbad = __any(seen.outside());
            if (RS) {
                vcol = a.vec[(size_t)n.seg * D + band * 32 + m];
                asm volatile("" : "+v"(vcol));             // waited for here: at each use the wait would drain the stores under way
            }
        }
        if (n.rows <= 0) continue;
        const bool slow = wbad || bad[u & 3];
        const v16f d = multiply_rows<1, false>(lds + (u & 1) * BUF + 3 * PLANE, w, m, kh, slow, wp, [&] {
            const int r = n.row0 + min(m, n.rows - 1);
            if (!SEL) return RowAt{a.dY + (size_t)(BOTH ? a.gather[r] : r) * a.ldd, 1.f};
            const int sl = a.ysel[r];
            return RowAt{selected_row(a, sl), selected_scale<RS>(a, r, sl)};
        });
        if (XSEL == 2) {
            int at = (4 * kh) * 512 + (band * 32 + m) * 4;
            asm volatile("" : "+v"(at));
            const unsigned char* const x = lds + 2 * BUF + (u & 1) * XROWS + at;
            float mine = 0.f;                              // lane m keeps the sum of the m-th of its half's 16 rows
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float p = group_sum<32>(d[v] * *reinterpret_cast<const float*>(x + (8 * (v >> 2) + (v & 3)) * 512));
                if (m == v) mine = p;
            }
            if (m < 16) dot_of[u & 3].band[band][8 * (m >> 2) + 4 * kh + (m & 3)] = mine;
        }
        store_rows<BOTH, RS>(d, a.dX + (BOTH ? 0 : (size_t)n.row0 * D) + band * 32 + m, n.rows, kh, D, row_of[u & 3].to, row_of[u & 3].s, vcol);
    }
}

template <bool GATHER, bool BOTH, bool RS, bool SEL, int XSEL>
__device__ __forceinline__ void bwd_gradient(const BwdArgs& a, unsigned char* lds, int* bad, int u0, int u1) {
    const int lane = threadIdx.x & 63, band = (threadIdx.x >> 6) & 3, m = lane & 31, kh = lane >> 5;
    // Transposing reads: the 16-column groups g and g + 4 of the 128 form a 32 x 32 block (see the bf16 backward); this
    // wavefront owns feature groups band and band + 4 of X and all four column blocks of dY.
    const int i16 = lane & 15, tg = (lane >> 4) & 1;
    // The first read's place is base; other column groups and the second four rows are XORs of it with constants
    // (row 8 kh + 4 t + q has swz 8 t + 2 q + kh, group b sits at piece 2 b), formed where they are used.
    const int q16 = i16 >> 2, base = (8 * kh + q16) * 256 + (((8 * tg + ((i16 & 3) >> 1)) ^ (2 * q16 + kh)) << 4) + (i16 & 1) * 8;
    v16f acc[4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;
    Units units(a.t, u0 >> 1, u1 >> 1);
    int cur_seg = -1, slot = a.t.chunk_slot[blockIdx.x] - 1;
    for (int u = u0 - 1; u <= u1; ++u) {
        __syncthreads();
        if (u < u0 || u > u1) continue;
        const Unit n = units.get(min(u, u1 - 1));
        const int seg = u < u1 ? n.seg : -2;
        if (seg != cur_seg) {
            if (cur_seg >= 0) {
                // (the lane's place is made opaque so that the 64 addresses are formed here and not kept across the loop)
                int at = (16 * band + 4 * kh) * D + (m & 15) + 64 * (m >> 4);
                asm volatile("" : "+v"(at));
                float* ps = a.part + (size_t)slot * SLOT + at;
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {         // block row 8 (v / 4) + 4 kh + v % 4: features 16 band + (0..15), then 64 further
                        ps[((v & 3) + 8 * ((v >> 2) & 1) + 64 * (v >> 3)) * D + 16 * b] = acc[b][v];
                        acc[b][v] = 0.f;
                    }
            }
            ++slot;
            cur_seg = seg;
        }
        if (u >= u1 || n.rows <= 0) continue;
        if (!bad[u & 3]) {
            int at = base;
            asm volatile("" : "+v"(at));                   // (not kept per group across the loop)
            const unsigned char* const Xt = lds + (u & 1) * BUF + (at ^ (band << 5));
            const unsigned char* const Xu = lds + (u & 1) * BUF + (at ^ (band << 5) ^ 128) + 1024;
            // The unit's products are summed on their own and then added to the running gradient: one rounding at the
            // gradient's magnitude per 32 rows (16 with the fp32 matrix instructions).
#pragma unroll
            for (int hb = 0; hb < 4; hb += 2) {            // two column blocks at a time
                v16f t0, t1;
#pragma unroll
                for (int v = 0; v < 16; ++v) t0[v] = t1[v] = 0.f;
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    bf16x8 x[3], y0[3], y1[3];
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const unsigned char* yt = lds + (u & 1) * BUF + (3 + q) * PLANE + s * 4096;
                        x[q] = tr8(Xt + q * PLANE + s * 4096, Xu + q * PLANE + s * 4096);
                        y0[q] = tr8(yt + (at ^ (hb << 5)), yt + (at ^ (hb << 5) ^ 128) + 1024);
                        y1[q] = tr8(yt + (at ^ ((hb + 1) << 5)), yt + (at ^ ((hb + 1) << 5) ^ 128) + 1024);
                    }
                    mfma_split2<0>(x, y0, t0, x, y1, t1);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    acc[hb][v] += t0[v];
                    acc[hb + 1][v] += t1[v];
                }
            }
        } else {
            constexpr int J = SEL ? 2 : 4;                 // rows in flight per half (the selector needs the registers)
            const int f = (m & 15) + 64 * (m >> 4);
            const int rm = n.row0 + min(m, n.rows - 1);
            const int gm = GATHER ? a.gather[rm] : 0, ym = SEL ? a.ysel[rm] : 0;    // of row m of the unit
            const float sm = XSEL == 2 ? a.yscale[a.num[rm]] : SEL && !XSEL ? selected_scale<RS>(a, rm, ym) : 1.f;      // (XSEL: of the X row)
#pragma unroll 1
            for (int k = 0; k < UNIT; k += 2 * J) {
                float x[J], y[J][4];
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const int q = min(k + 2 * j + kh, n.rows - 1), r = n.row0 + q, g = GATHER ? __shfl(gm, q) : r;
                    const float* const yp = SEL ? selected_row(a, __shfl(ym, q)) : a.dY + (size_t)(BOTH ? g : r) * a.ldd;
                    const float s = SEL ? __shfl(sm, q) : 1.f;
                    x[j] = input_row<XSEL>(a, g)[16 * band + f] * (XSEL == 2 ? s : 1.f);
#pragma unroll
                    for (int b = 0; b < 4; ++b) y[j][b] = yp[f + 16 * b] * (XSEL ? 1.f : s);
                }
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const bool ok = k + 2 * j + kh < n.rows;
#pragma unroll
                    for (int b = 0; b < 4; ++b) acc[b] = mfma32(ok ? x[j] : 0.f, ok ? y[j][b] : 0.f, acc[b]);
                }
            }
        }
    }
}

// GATHER: X rows through the list; BOTH: dY rows and dXrow rows as well; SEL: dY rows through the row selector; XSEL: X rows from two tensors
template <bool GATHER, bool BOTH, bool RS, bool SEL = false, int XSEL = 0>
__global__ __launch_bounds__(768) __attribute__((amdgpu_waves_per_eu(3, 3))) void typed_linear_split_bwd_kernel(BwdArgs a) {
    static_assert(!(BOTH && (RS || SEL)) && (GATHER || !BOTH) && (!XSEL || (GATHER && SEL && !RS)), "combinations the layers use");
    extern __shared__ __align__(16) unsigned char lds[];   // [2] plane buffers, [2][8][32] float4 vector sums
    __shared__ int bad[4];
    __shared__ __align__(16) RowOf row_of[4];
    __shared__ DotOf dot_of[XSEL == 2 ? 4 : 1];
    const int u0 = 2 * a.t.chunk_tile[blockIdx.x], u1 = 2 * a.t.chunk_tile[blockIdx.x + 1];
    if (threadIdx.x < 4) bad[threadIdx.x] = 0;
    __syncthreads();
    if (u0 >= u1) return;
    if (threadIdx.x < 256) bwd_multiply<GATHER, BOTH, RS, SEL, XSEL>(a, lds, row_of, dot_of, bad, u0, u1);
    else if (threadIdx.x < 512) bwd_gradient<GATHER, BOTH, RS, SEL, XSEL>(a, lds, bad, u0, u1);
    else bwd_load<GATHER, BOTH, RS, SEL, XSEL>(a, lds, reinterpret_cast<float4*>(lds + 2 * BUF), row_of, dot_of, bad, u0, u1);
}

TileArgs tile_args(const TileList& t) { return TileArgs{t.tile_seg, t.tile_row0, t.tile_row1, t.chunk_tile, t.chunk_slot}; }

template <bool SCATTER>
rgnn_status_t launch_fwd(const TypedLinearArgs& a, const TileList& t, hipStream_t st) {
    const size_t lds = 2 * 3 * PLANE + 2 * STAGE;
    auto kern = typed_linear_split_fwd_kernel<SCATTER>;
    RGNN_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds));
    KernelTimer kt(st, a.label ? a.label : "typed_linear_fwd");
    hipLaunchKernelGGL(kern, dim3(t.num_chunks), dim3(512), lds, st,
                       FwdArgs{tile_args(t), a.X, a.gather, a.W, a.Y, a.y_stride * D});
    RGNN_HIP(hipGetLastError());
    return RGNN_OK;
}
template <bool GATHER, bool BOTH, bool RS, bool SEL = false, int XSEL = 0>
rgnn_status_t launch_bwd(const TypedLinearBwdArgs& a, const TileList& t, hipStream_t st) {
    const size_t lds = 2 * BUF + (XSEL == 2 ? 2 * XROWS : 2 * 256 * (int)sizeof(float4));
    auto kern = typed_linear_split_bwd_kernel<GATHER, BOTH, RS, SEL, XSEL>;
    RGNN_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds));
    KernelTimer kt(st, a.label ? a.label : "typed_linear_bwd");
    hipLaunchKernelGGL(kern, dim3(t.num_chunks), dim3(768), lds, st,
                       BwdArgs{tile_args(t), a.X, a.gather, a.W, a.dY, a.dy_stride * D, a.dXrow, a.rowscale, a.vec, a.part, a.ysel, a.dY_alt,
                               a.ds_yscale, a.yscale, a.X2, a.rowdot, a.num});
    RGNN_HIP(hipGetLastError());
    return RGNN_OK;
}

}  // namespace

rgnn_status_t typed_linear_split_fwd(const TypedLinearArgs& a, hipStream_t st) {
    const TileList& t = *a.tiles;
    if (t.num_tiles == 0) return RGNN_OK;
    if (!a.gather || a.accumulate || a.vec || a.relu || a.X2)
        RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear forward: the split product is built for gathered rows, without accumulate / vec / activation");
    return a.scatter_out ? launch_fwd<true>(a, t, st) : launch_fwd<false>(a, t, st);
}

rgnn_status_t typed_linear_split_bwd(const TypedLinearBwdArgs& a, hipStream_t st) {
    const TileList& t = *a.tiles;
    const bool g = a.gather != nullptr, dg = g && a.dy_gathered, sc = g && a.scatter_dx, rs = a.rowscale != nullptr;
    if (a.X2) {
        if (!g || dg || sc || rs || !a.ysel || a.dY_alt || a.vec || a.ds_yscale || a.hcoef || a.dy_stride != 1)
            RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear backward: two input tensors go with gathered X, a list of the dY rows and scales at most");
        if (t.num_tiles == 0) return RGNN_OK;
        return a.yscale ? launch_bwd<true, false, false, true, 2>(a, t, st) : launch_bwd<true, false, false, true, 1>(a, t, st);
    }
    if (a.ysel && (dg || !g || rs || a.dy_stride != 1 || a.hcoef || !a.dY_alt || (a.ds_yscale ? !a.vec || a.yscale : a.vec != nullptr)))
        RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear backward: the row selector needs gathered X, ungathered dY, and vec with the (rowscale, scale) pairs or neither; no heads at width 128");
    if (dg != sc) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear backward: dY gathered and dXrow scattered must go together");
    if (rs && (dg || !g || !a.vec)) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed linear backward: rowscale needs vec, gathered X and ungathered dY");
    if (t.num_tiles == 0) return RGNN_OK;
    if (a.ysel) return a.ds_yscale ? launch_bwd<true, false, true, true>(a, t, st) : launch_bwd<true, false, false, true>(a, t, st);
    if (rs) return launch_bwd<true, false, true>(a, t, st);
    if (dg) return launch_bwd<true, true, false>(a, t, st);
    if (g) return launch_bwd<true, false, false>(a, t, st);
    return launch_bwd<false, false, false>(a, t, st);
}

}  // namespace rgnn
