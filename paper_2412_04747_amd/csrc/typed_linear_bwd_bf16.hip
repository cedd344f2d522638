// Backward of the typed linear layer on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16), width 128, X and dY rows in
// bf16, fp32 accumulation:   dXrow[i] = dY[i] W[seg]^T   and   part[slot] = sum over the chunk's rows of X[g(i)]^T dY[i]
// in one pass over the rows (one weight, or two weights whose gradient rows lie side by side:
// dXrow = dY0 W0^T + dY1 W1^T, part = (X^T dY0, X^T dY1)).
//
// Bound by HBM: the two products together need a tenth of the matrix cores' rate at the speed the rows arrive.  As two
// kernels the dY rows were read twice (and for two weights the X rows twice, the dXrow rows written twice and summed
// later).  14.5M pairs (single-edge rows through the selector, 500 relations): 1.33 + 1.40 ms as two kernels, now 1.84 ms
// (11.1 GB, 6.0 TB/s); 5.4M pairs with two weights: 2.12 ms as four kernels, now 1.10 ms (5.5 GB, 5.0 TB/s).
//
// A workgroup of eight wavefronts takes a chunk of 64-row tiles.  A tile's X and dY rows are brought to registers one tile
// ahead and written to LDS row-major.  dXrow^T = W dY^T takes W's rows and the dY rows as its operands straight from LDS
// (each wavefront forms 32 rows x 32 input features); the weight gradient contracts over rows, and its operands (eight consecutive rows of a feature) come from the same tiles through the transposing LDS read
// ds_read_b64_tr_b16, which hands lane i of 16 the i-th column of four rows.
// LDS: 16-byte piece c of row r sits at piece c ^ swz(r).  swz takes 16 different values over 16 consecutive rows, so the
// row operands (16 lanes, 16 rows, one piece) fall on different banks; over four rows it steps by 2, so the four rows of
// a transposing read fall on different pairs of pieces, and the second group of 16 lanes reads features 64 further (eight
// pieces), on the other half of the banks.
#include "rgnn_internal.h"
#include "device_utils.h"

namespace rgnn {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

struct BwdArgs {
    const int32_t* tile_seg;
    const int32_t* tile_row0;
    const int32_t* tile_row1;
    const int32_t* chunk_tile;
    const int32_t* chunk_slot;
    const bf16_t* X;
    const int32_t* gather;
    const bf16_t* dY;
    int ldd;                 // elements from one row of dY to the next
    const int32_t* ysel;
    const bf16_t* dY_alt;
    const float* yscale;
    const int32_t* sum_ptr;  // PAIRS
    const int32_t* sum_row;
    const bf16_t* sum_rows;
    const void* W[2];
    void* dX;
    float* part;
};


// eight bf16 (four packed pairs) times s, rounded to nearest even again
__device__ __forceinline__ rgnn_v4u scale8(rgnn_v4u x, float s) {
    rgnn_v4u y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = bf16_pack2(__uint_as_float(x[e] << 16) * s, __uint_as_float(x[e] & 0xFFFF0000u) * s);
    return y;
}

//   NB     weights (dY rows are NB * 128 wide)        WPL    planes of W: 1 = bf16, 2 = fp32 split into hi + lo
//   GATHER X rows through the gather list             BOTH   dY rows are read and dXrow rows written through it as well
//   SEL    row i of dY is dY[ysel[i]], or dY_alt[ysel[i] & 0x7FFFFFFF] when the top bit of ysel[i] is set; with yscale it is
//          multiplied by yscale[i] (and rounded to bf16 again) on its way into LDS
//   DX32   dXrow is fp32, ACC: and added to           otherwise bf16
//   PAIRS  with BOTH and DX32: dXrow row n also gets the sum of the rows sum_row[sum_ptr[n] .. sum_ptr[n + 1]) of sum_rows (HGT: the query's
//          part of dX and the sum over the node's pairs).  A lane adds its 16 columns of its row, two rows at a time, the list two tiles ahead.
//          As a walk of its own that read the query's part again: 2M nodes, 5.4M pairs 408 + 670 us, so 829 in
//          chunks that weigh alike (chunk_tiles), 862 in chunks of as many tiles; where node types differ in their pairs, 2M nodes, 4.5M pairs,
//          406 + 617, 783 and 1079.  (Whole rows added by the threads
//          that load a tile, and handed over through LDS, need 25 registers more than two workgroups per compute unit leave: 968 for the 862.)
template <int NB, int WPL, bool GATHER, bool BOTH, bool SEL, bool DX32, bool ACC, bool PAIRS = false>
__device__ __forceinline__ void bwd_tiles(const BwdArgs& a) {
    static_assert(!(SEL && BOTH) && (GATHER || !BOTH) && (DX32 || !ACC) && (NB == 1 || !SEL) && (!PAIRS || (BOTH && DX32)), "combinations the layers use");
    constexpr int D = 128, TILE = 64 * 2 * D;             // bytes of a 64-row tile
    constexpr int SLOT = NB * D * D;
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int WT = 128 * 2 * D;                       // bytes of a plane of W
    unsigned char* const Wl = lds;                        // [NB][WPL][128][256]
    unsigned char* const Xt = lds + NB * WPL * WT;        // [64][256]
    unsigned char* const Yt = Xt + TILE;                  // [NB][64][256]
    unsigned char* const St = Yt + NB * TILE;             // [64][256]  bf16 dXrow tile on its way out
    int* const gidx = reinterpret_cast<int*>(St);         // DX32: [64] destination rows instead
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = lane & 31, kh = lane >> 5;
    // rows in and out: 16 lanes per row, two rows per thread
    const int lc = tid & 15, lr = tid >> 4;
    const int io = lr * 256 + ((lc ^ swz(lr)) << 4);
    // dXrow block of this wavefront: 32 rows x 32 input features
    const int rb = wave & 1, ob = wave >> 1;
    const int yrow = (rb * 32 + m) * 256, wrow = (ob * 32 + m) * 256, ysw = (kh ^ swz(m)) << 4;
    // weight-gradient blocks: features 16 fb + (0..15) and 64 further x two column blocks per weight, laid out alike
    const int fb = wave & 3, cb = (wave >> 2) * 2;
    const int ti16 = lane & 15, tg = (lane >> 4) & 1;
    int xoff[2], yoff[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int r = 8 * kh + 4 * t + (ti16 >> 2), piece = (ti16 & 3) >> 1, half = (ti16 & 1) * 8;
        xoff[t] = r * 256 + (((2 * (fb + 4 * tg) + piece) ^ swz(r)) << 4) + half;
#pragma unroll
        for (int x = 0; x < 2; ++x) yoff[x][t] = r * 256 + (((2 * (cb + x + 4 * tg) + piece) ^ swz(r)) << 4) + half;
    }
    v16f acc[NB][2];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[nb][x][v] = 0.f;
    const int t0 = a.chunk_tile[blockIdx.x], t1 = a.chunk_tile[blockIdx.x + 1];
    rgnn_v4u xr[2], yr[NB][2];
    int gi[2], gy[2], gcur[2];
    float sc[2] = {1.f, 1.f}, scc[2] = {1.f, 1.f};
    TileTable tt(a.tile_seg, a.tile_row0, a.tile_row1, t0, t1);
    auto fetch_idx = [&](int ti) {
        const int l = tt.lane_of(ti), row0 = tt.row0_at(l), row1 = tt.row1_at(l);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int row = min(row0 + lr + 32 * k, row1 - 1);
            gi[k] = GATHER ? a.gather[row] : row;
            gy[k] = SEL ? a.ysel[row] : BOTH ? gi[k] : row;
            if (SEL && a.yscale) sc[k] = a.yscale[row];
        }
    };
    auto fetch = [&]() {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            xr[k] = *reinterpret_cast<const rgnn_v4u*>(a.X + (size_t)gi[k] * D + lc * 8);
            const bf16_t* y = SEL && gy[k] < 0 ? a.dY_alt : a.dY;
            y += (size_t)(SEL ? gy[k] & 0x7FFFFFFF : gy[k]) * a.ldd + lc * 8;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) yr[nb][k] = *reinterpret_cast<const rgnn_v4u*>(y + nb * D);
            gcur[k] = gi[k];
            scc[k] = sc[k];
        }
    };
    if (t0 >= t1) return;
    // PAIRS: list ends and first four entries of the lane's row rb * 32 + m of this tile, list ends one tile on, node two tiles on
    int pb = 0, pe = 0, p0 = 0, p1 = 0, p2 = 0, p3 = 0, pbn = 0, pen = 0, node = 0;
    auto node_of = [&](int ti) {
        const int l = tt.lane_of(ti);
        return a.gather[min(tt.row0_at(l) + rb * 32 + m, tt.row1_at(l) - 1)];
    };
    auto pair_at = [&](int p, int e) { return a.sum_row[max(min(p, e - 1), 0)]; };
    if (PAIRS) {
        node = node_of(t0);
        pb = a.sum_ptr[node]; pe = a.sum_ptr[node + 1];
        node = node_of(min(t0 + 1, t1 - 1));
        pbn = a.sum_ptr[node]; pen = a.sum_ptr[node + 1];
        node = node_of(min(t0 + 2, t1 - 1));
        p0 = pair_at(pb, pe); p1 = pair_at(pb + 1, pe); p2 = pair_at(pb + 2, pe); p3 = pair_at(pb + 3, pe);
    }
    fetch_idx(t0);
    fetch();
    fetch_idx(min(t0 + 1, t1 - 1));
    int cur_seg = -1, slot = a.chunk_slot[blockIdx.x] - 1;
    for (int ti = t0; ti <= t1; ++ti) {
        const int tl = tt.lane_of(min(ti, t1 - 1)), seg = ti < t1 ? tt.seg_at(tl) : -2;
        if (seg != cur_seg) {
            if (cur_seg >= 0) {
                // (the lane's place is made opaque so that the addresses are formed here and not kept across the loop)
                int at = (16 * fb + 4 * kh) * D + 16 * cb + (m & 15) + 64 * (m >> 4);
                asm volatile("" : "+v"(at));
                float* ps = a.part + (size_t)slot * SLOT + at;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
#pragma unroll
                        for (int v = 0; v < 16; ++v) {     // block row 8 (v / 4) + 4 kh + v % 4: features 16 fb + (0..15), then 64 further
                            ps[nb * D * D + ((v & 3) + 8 * ((v >> 2) & 1) + 64 * (v >> 3)) * D + 16 * x] = acc[nb][x][v];
                            acc[nb][x][v] = 0.f;
                        }
            }
            if (ti == t1) break;
            ++slot;
            cur_seg = seg;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                unsigned char* const wl = Wl + nb * WPL * WT;
#pragma unroll
                for (int k = 0; k < 4; ++k) {             // 32 rows of W per pass, 16 pieces each
                    const size_t at = (size_t)seg * D * D + (size_t)(lr + 32 * k) * D + lc * 8;
                    if (WPL == 1) {
                        *reinterpret_cast<rgnn_v4u*>(wl + io + k * 32 * 256) =
                            *reinterpret_cast<const rgnn_v4u*>(static_cast<const bf16_t*>(a.W[nb]) + at);
                    } else {
                        float x[8];
                        load_cols(static_cast<const float*>(a.W[nb]) + at, x);
                        rgnn_v4u hi, lo;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            hi[e] = bf16_pack2(x[2 * e], x[2 * e + 1]);
                            lo[e] = bf16_pack2(x[2 * e] - __uint_as_float(hi[e] << 16), x[2 * e + 1] - __uint_as_float(hi[e] & 0xFFFF0000u));
                        }
                        *reinterpret_cast<rgnn_v4u*>(wl + io + k * 32 * 256) = hi;
                        *reinterpret_cast<rgnn_v4u*>(wl + (WPL - 1) * WT + io + k * 32 * 256) = lo;
                    }
                }
            }
        }
        const int row0 = tt.row0_at(tl), rows = tt.row1_at(tl) - row0;
        int gout[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const bool ok = lr + 32 * k < rows;            // rows past the end of the tile count as zeros
            const rgnn_v4u z = {0u, 0u, 0u, 0u};
            *reinterpret_cast<rgnn_v4u*>(Xt + io + k * 32 * 256) = ok ? xr[k] : z;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                rgnn_v4u y = yr[nb][k];
                if (SEL && a.yscale) y = scale8(y, scc[k]);
                *reinterpret_cast<rgnn_v4u*>(Yt + nb * TILE + io + k * 32 * 256) = ok ? y : z;
            }
            gout[k] = gcur[k];
            if (DX32 && BOTH && lc == 0) gidx[lr + 32 * k] = gcur[k];
        }
        __syncthreads();   // the tile is complete
        const int sb = pb, se = pe, s0 = p0, s1 = p1, s2 = p2, s3 = p3;
        if (PAIRS) {
            pb = pbn; pe = pen;
            p0 = pair_at(pb, pe); p1 = pair_at(pb + 1, pe); p2 = pair_at(pb + 2, pe); p3 = pair_at(pb + 3, pe);
            pbn = a.sum_ptr[node]; pen = a.sum_ptr[node + 1];
            node = node_of(min(ti + 3, t1 - 1));
        }
        // (unconditional, past the end the last tile again: were the loads skipped on some path, the waits for the rows would
        // have to drain the stores issued after them as well)
        fetch();
        fetch_idx(min(ti + 2, t1 - 1));
        v16f d;
#pragma unroll
        for (int v = 0; v < 16; ++v) d[v] = 0.f;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int at = ysw ^ (s << 5);
                const bf16x8 by = *reinterpret_cast<const bf16x8*>(Yt + nb * TILE + yrow + at);
#pragma unroll
                for (int pl = 0; pl < WPL; ++pl)
                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(Wl + (nb * WPL + pl) * WT + wrow + at), by, d, 0, 0, 0);
            }
        // d[v] = dXrow[row rb * 32 + m][feature ob * 32 + 8 (v / 4) + 4 kh + v % 4]
        if (PAIRS) {
            // two rows at a time, 16 columns of each to a lane
            auto add2 = [&](int i0, int i1, bool two) {
                uint2 x[2][4];
                const bf16_t* const r0 = a.sum_rows + (size_t)i0 * D + ob * 32 + 4 * kh;
                const bf16_t* const r1 = a.sum_rows + (size_t)i1 * D + ob * 32 + 4 * kh;
#pragma unroll
                for (int q = 0; q < 4; ++q) x[0][q] = *reinterpret_cast<const uint2*>(r0 + 8 * q);
#pragma unroll
                for (int q = 0; q < 4; ++q) x[1][q] = *reinterpret_cast<const uint2*>(r1 + 8 * q);
#pragma unroll
                for (int y = 0; y < 2; ++y)
                    if (y == 0 || two) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            d[4 * q] += __uint_as_float(x[y][q].x << 16); d[4 * q + 1] += __uint_as_float(x[y][q].x & 0xFFFF0000u);
                            d[4 * q + 2] += __uint_as_float(x[y][q].y << 16); d[4 * q + 3] += __uint_as_float(x[y][q].y & 0xFFFF0000u);
                        }
                    }
            };
            if (sb < se) add2(s0, s1, sb + 1 < se);
            if (sb + 2 < se) add2(s2, s3, sb + 3 < se);
            for (int p = sb + 4; p < se; p += 2) add2(a.sum_row[p], pair_at(p + 1, se), p + 1 < se);
        }
        if (DX32) {
            if (rb * 32 + m < rows) {
                const size_t r = BOTH ? (size_t)gidx[rb * 32 + m] : (size_t)(row0 + rb * 32 + m);
                float* o = static_cast<float*>(a.dX) + r * D + ob * 32 + 4 * kh;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float4 y = make_float4(d[4 * q], d[4 * q + 1], d[4 * q + 2], d[4 * q + 3]);
                    float4* p = reinterpret_cast<float4*>(o + 8 * q);
                    if (ACC) {
                        const float4 old = *p;
                        y.x += old.x; y.y += old.y; y.z += old.z; y.w += old.w;
                    }
                    *p = y;
                }
            }
        } else {
            const int sw = swz(m);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<uint2*>(St + yrow + (((ob * 4 + q) ^ sw) << 4) + 8 * kh) =
                    make_uint2(bf16_pack2(d[4 * q], d[4 * q + 1]), bf16_pack2(d[4 * q + 2], d[4 * q + 3]));
        }
        __builtin_amdgcn_sched_barrier(0);      // the dXrow registers are free before the weight-gradient operands are read
        // A tile's products are summed on their own and then added to the running gradient: one rounding at the gradient's
        // magnitude per 64 rows instead of four.  In one chain of matrix instructions the error of dW grows with the chunk: 6M
        // rows of 4 relations 7.0e-7 against 64 bits, 3M rows with two weights 7.0e-7; so: 2.7e-7 and 2.8e-7.
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            v16f t[2];
#pragma unroll
            for (int v = 0; v < 16; ++v) t[0][v] = t[1][v] = 0.f;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const bf16x8 ax = tr8(Xt + xoff[0] + s * 4096, Xt + xoff[1] + s * 4096);
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    const unsigned char* y = Yt + nb * TILE + s * 4096;
                    t[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ax, tr8(y + yoff[x][0], y + yoff[x][1]), t[x], 0, 0, 0);
                }
                if (s & 1) __builtin_amdgcn_sched_barrier(0);      // (operands of two steps at a time)
            }
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[nb][x][v] += t[x][v];
        }
        __syncthreads();   // operand reads are done, the result tile is complete
        if (!DX32) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int r = lr + 32 * k;
                if (r < rows) {
                    const size_t to = BOTH ? (size_t)gout[k] : (size_t)(row0 + r);
                    __builtin_nontemporal_store(*reinterpret_cast<const rgnn_v4u*>(St + io + k * 32 * 256),
                                                reinterpret_cast<rgnn_v4u*>(static_cast<bf16_t*>(a.dX) + to * D + lc * 8));
                }
            }
        }
    }
}

// One weight in bf16: 128 registers and 80 KB of LDS leave room for two workgroups per compute unit, so that one loads
// while the other multiplies; two weights (or one split into two planes) take twice the room for W and run alone.
template <bool GATHER, bool BOTH, bool SEL, bool DX32, bool ACC, bool PAIRS = false>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4))) void typed_linear_bwd_bf16_kernel(BwdArgs a) {
    bwd_tiles<1, 1, GATHER, BOTH, SEL, DX32, ACC, PAIRS>(a);
}
template <int NB, int WPL, bool GATHER, bool BOTH, bool SEL, bool DX32, bool ACC>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void typed_linear_bwd_bf16_big_kernel(BwdArgs a) {
    bwd_tiles<NB, WPL, GATHER, BOTH, SEL, DX32, ACC>(a);
}

// nb weights in wpl planes each
template <typename K>
rgnn_status_t launch(K kern, const TypedLinearBwdBf16Args& a, int nb, int wpl, hipStream_t st) {
    const size_t lds = (size_t)(2 + nb) * 64 * 256 + (size_t)nb * wpl * 128 * 256;
    RGNN_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(kern), lds));
    const TileList& t = *a.tiles;
    BwdArgs b{t.tile_seg, t.tile_row0, t.tile_row1, t.chunk_tile, t.chunk_slot, static_cast<const bf16_t*>(a.X), a.gather,
              static_cast<const bf16_t*>(a.dY), a.dy_stride * 128, a.ysel, static_cast<const bf16_t*>(a.dY_alt), a.yscale,
              a.sum_ptr, a.sum_row, static_cast<const bf16_t*>(a.sum_rows), {a.W, a.W2}, a.dXrow, a.part};
    KernelTimer kt(st, a.label);
    hipLaunchKernelGGL(kern, dim3(t.num_chunks), dim3(512), lds, st, b);
    RGNN_HIP(hipGetLastError());
    return RGNN_OK;
}

}  // namespace

rgnn_status_t typed_linear_bwd_bf16(int d, const TypedLinearBwdBf16Args& a, hipStream_t st) {
    if (d != 128) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_bwd_bf16: width %d not supported (128)", d);
    if (a.tiles->num_tiles > 0) {
        const bool both = a.both_gathered != 0, sel = a.ysel != nullptr;
        if (both && !a.gather) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_bwd_bf16: rows gathered on both sides need a gather list");
        if (!a.gather) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_bwd_bf16: built for gathered X rows");
        if (sel && (both || !a.dY_alt || a.dx_f32 || a.dy_stride != 1 || a.W2 || !a.w_bf16))
            RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_bwd_bf16: the row selector is built for one bf16 weight, ungathered dY and bf16 result rows");
        if (a.accumulate && !(both && a.dx_f32)) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_bwd_bf16: accumulation is built for fp32 rows gathered on both sides");
        if (a.sum_rows && (!both || !a.dx_f32 || a.W2 || !a.w_bf16 || !a.sum_ptr || !a.sum_row))
            RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_bwd_bf16: rows are added for one bf16 weight, fp32 rows gathered on both sides");
        if (a.W2) {
            if (both || a.dx_f32 || !a.w_bf16 || a.dy_stride != 2) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_bwd_bf16: two weights are built in bf16, for gradient rows side by side and bf16 result rows");
            RGNN_TRY(launch(typed_linear_bwd_bf16_big_kernel<2, 1, true, false, false, false, false>, a, 2, 1, st));
        } else if (!a.w_bf16) {
            if (both || a.dx_f32) RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_bwd_bf16: an fp32 weight is built for ungathered dY and bf16 result rows");
            RGNN_TRY(launch(typed_linear_bwd_bf16_big_kernel<1, 2, true, false, false, false, false>, a, 1, 2, st));
        } else if (sel) {
            RGNN_TRY(launch(typed_linear_bwd_bf16_kernel<true, false, true, false, false>, a, 1, 1, st));
        } else if (a.sum_rows) {
            if (a.accumulate) RGNN_TRY(launch(typed_linear_bwd_bf16_kernel<true, true, false, true, true, true>, a, 1, 1, st));
            else RGNN_TRY(launch(typed_linear_bwd_bf16_kernel<true, true, false, true, false, true>, a, 1, 1, st));
        } else if (both && a.dx_f32 && a.accumulate) {
            RGNN_TRY(launch(typed_linear_bwd_bf16_kernel<true, true, false, true, true>, a, 1, 1, st));
        } else if (both && a.dx_f32) {
            RGNN_TRY(launch(typed_linear_bwd_bf16_kernel<true, true, false, true, false>, a, 1, 1, st));
        } else if (both) {
            RGNN_TRY(launch(typed_linear_bwd_bf16_kernel<true, true, false, false, false>, a, 1, 1, st));
        } else if (!a.dx_f32) {
            RGNN_TRY(launch(typed_linear_bwd_bf16_kernel<true, false, false, false, false>, a, 1, 1, st));
        } else {
            RGNN_FAIL(RGNN_EUNSUPPORTED, "typed_linear_bwd_bf16: this combination is not built");
        }
    }
    return typed_linear_slot_reduce(*a.tiles, a.part, d * d, a.W2 ? d * d : 0, a.dW, a.dW2, st, a.sums);
}

}  // namespace rgnn
