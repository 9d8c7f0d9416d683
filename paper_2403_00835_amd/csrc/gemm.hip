// Weight-streaming GEMM of libcllm.so on gfx950 (CDNA4): the products of a Jacobi iteration
// (QKV, O, gate/up, down, LM head) with their fused epilogues, and the fp32-output product of
// the training loss head.
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

#include "device.h"
#include "launch.h"

namespace cllm {

// ------------------------------------------------------------------------------------------
// Weight-streaming GEMM:  Y[rows x N] = A[rows x K] * W^T,  W packed in 1 KiB tiles.
//
// Packed layout: tile (t, s) covers weight rows 16t .. 16t+15 (after the per-GEMM row order)
// and K indices s*KSTEP .. s*KSTEP+KSTEP-1; lane l's 16 bytes are row 16t + l%16, K indices
// s*KSTEP + (l/16)*VEC .. +VEC. Tiles are stored k-step major: tile (t, s) at index s * T + t
// (T tiles per k-step), so the tiles every workgroup reads for one k-step are one contiguous
// region (measured 1-7% faster streaming than row blocks contiguous over s).
//
// A workgroup of 8 waves owns NT consecutive tiles (16*NT output columns) for all rows; wave w
// takes k-steps w, w+8, w+16, ... and accumulates them in order with MFMA; the 8 partial tiles
// are then summed in a fixed tree ((w0+w4)+(w2+w6))+((w1+w5)+(w3+w7)). Weights are read once,
// straight into registers (no LDS); the activation rows (a few KiB, L2-resident) are re-read.
// In bf16 the activations are fp32 values split into hi and lo bf16 planes, and each k-step runs
// one MFMA per plane against the same weight tile: products are exact in fp32, so the operand
// keeps 16 significant bits instead of bf16's 8.
//
// Products that follow an RMSNorm take the operand x (.) g written by the producer of x and
// scale each output row by 1/sqrt(mean(x^2) + eps), reduced from the producer's per-16-column
// sums of squares.
// ------------------------------------------------------------------------------------------

enum Epi { E_QKV = 0, E_RESID = 1, E_SWIGLU = 2, E_ARGMAX = 3, E_LOGITS = 4 };

template <Prec P, int NT, int RG>
struct Stage {  // operands of one k-step
    u32x4 b[NT];                      // weight tiles
    u32x4 a[PrecT<P>::PLANES][RG];    // activation rows (hi, lo planes for bf16)
};

// Loads of one k-step s (callers clamp s into [0, Ks), so every load is issued and the compiler
// can count outstanding loads exactly). Tiles past the last one (a ragged last workgroup) load
// the last tile again; their columns are never written. SHARED: the weight tiles are read by
// several workgroups (the row tiles of one column group), so they are loaded as ordinary
// (cached) loads; otherwise they are streamed (nontemporal: read once, not kept in the caches).
template <Prec P, int NT, int RG, bool SHARED>
__device__ __forceinline__ void gemm_load(Stage<P, NT, RG> &st, const GemmParams &p, int t0, int rg0, int s, int lane) {
    using PT = PrecT<P>;
    using T = typename PT::T;
    const int tiles = p.cols >> 4;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const u32x4 *src =
            reinterpret_cast<const u32x4 *>(p.W + ((size_t)s * tiles + min(t0 + j, tiles - 1)) * kTileBytes) + lane;
        st.b[j] = SHARED ? *src : __builtin_nontemporal_load(src);
    }
    const T *A = reinterpret_cast<const T *>(p.A);
    const int ks_a = p.lda / PT::KSTEP;
#pragma unroll
    for (int pl = 0; pl < PT::PLANES; ++pl)
#pragma unroll
        for (int r = 0; r < RG; ++r)
            st.a[pl][r] = *reinterpret_cast<const u32x4 *>(A + pl * act_plane(p.rr.cap, p.lda) +
                                                          ((size_t)((rg0 + r) * ks_a + s) * kWave + lane) * PT::VEC);
}

// MFMAs of one k-step: every hi-plane product, then every lo-plane product (bf16).
template <Prec P, int NT, int RG>
__device__ __forceinline__ void gemm_compute(const Stage<P, NT, RG> &st, f32x4 (&acc)[RG][NT]) {
#pragma unroll
    for (int pl = 0; pl < PrecT<P>::PLANES; ++pl)
#pragma unroll
        for (int r = 0; r < RG; ++r)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[r][j] = mfma_kstep<P>(st.a[pl][r], st.b[j], acc[r][j]);
}

__device__ __forceinline__ float silu(float x) { return x / (1.0f + expf(-x)); }

// Row factor 1/sqrt(mean(x^2) + eps) of the rows [row0, row0 + ROWS) from the producer's
// per-16-column sums of squares (layout [row][T], T a multiple of 4). 32 threads per row each add
// a contiguous run of q = 4 * ceil(T/128) partials in order (16-byte reads), then a fixed xor tree
// over the row's 32 threads; the scheme depends only on T, never on the number of rows. The
// first two vectors of the first row pass are requested early by row_factor_preload. The caller's
// next barrier publishes s_inv.
template <int W>
__device__ __forceinline__ void row_factor_preload(const GemmParams &p, int row0, int tid, f32x4 (&sq_pre)[2]) {
    const int sq_part = tid & 31, sq_q = ((p.T + 127) >> 7) << 2;
    const float *src = p.ssq + (size_t)(row0 + (tid >> 5)) * p.T;
#pragma unroll
    for (int i = 0; i < 2; ++i)  // clamped, unconditional
        sq_pre[i] = *reinterpret_cast<const f32x4 *>(src + min(sq_part * sq_q + 4 * i, p.T - 4));
}

template <int W, int ROWS>
__device__ __forceinline__ void row_factor_reduce(const GemmParams &p, int row0, int tid, const f32x4 (&sq_pre)[2],
                                                  float *s_inv) {
    constexpr int RPP = W * kWave / 32;  // rows per pass
    static_assert(ROWS % RPP == 0, "row passes cover the row groups");
    const int sq_part = tid & 31, sq_q = ((p.T + 127) >> 7) << 2;
    for (int pass = 0; pass < ROWS / RPP; ++pass) {
        const int row = pass * RPP + (tid >> 5);
        const float *src = p.ssq + (size_t)(row0 + row) * p.T;
        float sum = 0.0f;
        for (int i0 = 0; i0 < sq_q; i0 += 8) {
            f32x4 v[2];
            if (pass == 0 && i0 == 0) {
                v[0] = sq_pre[0];
                v[1] = sq_pre[1];
            } else {
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    v[i] = *reinterpret_cast<const f32x4 *>(src + min(sq_part * sq_q + i0 + 4 * i, p.T - 4));
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i0 + i < sq_q && sq_part * sq_q + i0 + i < p.T) sum += v[i >> 2][i & 3];
        }
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 32);
        if (sq_part == 0) s_inv[row] = 1.0f / sqrtf(sum / (float)p.K + p.eps);
    }
}

// Epilogues of a finished ROWS x COLS output tile in s_tile (row stride COLS + 1) for rows
// [row0, row0 + ROWS) of the iteration (m of them live) and column workgroup wg of width COLS
// (columns at or past p.cols, in a ragged last workgroup, are dropped); s_red is scratch of at
// least ROWS x COLS floats.
template <Prec P, int NT, int RG, int EP, int W>
__device__ __forceinline__ void gemm_epilogue(const GemmParams &p, float *s_tile, float *s_red, int row0, int m, int wg,
                                              int tid, int lane, int w) {
    using T = typename PrecT<P>::T;
    constexpr int ROWS = 16 * RG, COLS = 16 * NT;
    const int t0 = wg * NT;
    if constexpr (EP == E_QKV) {
        // Packed columns -> (section, head, dim). Tile b of a head holds dims [8b, 8b+8) and
        // their rotate-half partners [hd/2+8b, hd/2+8b+8): column o of the tile and column o ^ 8
        // are partners, so every tile is complete for RoPE and a workgroup may own any number
        // of tiles.
        const int hd = p.hd, d = p.d, h2 = hd >> 1;
        for (int idx = tid; idx < ROWS * COLS; idx += W * kWave) {
            const int row = idx / COLS, pc = idx % COLS;
            const int R = t0 * 16 + pc;  // packed row index
            if (row >= m || R >= p.cols) continue;
            const int sec = R / d, within = R % d, head = within / hd;
            const int q = within % hd, b = q >> 4, o = q & 15;
            const int dim = o < 8 ? 8 * b + o : h2 + 8 * b + (o - 8);
            const int partner = pc ^ 8;
            const RowInfo ri = p.rr.rows[row0 + row];
            const int pos = ri.pos;
            const size_t kvo = (size_t)p.rr.tab->seq[ri.b] * p.kv_seq;  // this row's sequence slot
            float x = s_tile[row * (COLS + 1) + pc];
            if (sec < 2) {
                const float y = s_tile[row * (COLS + 1) + partner];
                const int j = dim < h2 ? dim : dim - h2;
                const float c = p.rcos[(size_t)pos * h2 + j], s = p.rsin[(size_t)pos * h2 + j];
                x = dim < h2 ? (x * c - y * s) : (x * c + y * s);
            }
            const T e = to_elem<P>(x);  // cached keys and values are rounded to the cache dtype
            if (sec == 0)
                put_act<P>(reinterpret_cast<T *>(p.Q), act_plane(p.rr.cap, d), act_idx<P>(row0 + row, head * hd + dim, d), x);
            else if (sec == 1)
                reinterpret_cast<T *>(p.Kc)[kvo + (size_t)head * p.ctx_alloc * hd + kcache_idx<P>(pos, dim, hd)] = e;
            else
                reinterpret_cast<T *>(p.Vt)[kvo + (size_t)head * p.ctx_alloc * hd + vcache_idx<P>(pos, dim, hd)] = e;
        }
    } else if constexpr (EP == E_RESID) {
        // X += Y over this workgroup's columns, then the per-16-column sums of squares of the
        // new rows (summed in column order) for the next RMSNorm.
        const int c0 = t0 * 16;
        float *s_sq = s_red;  // ROWS x COLS
        for (int idx = tid; idx < ROWS * COLS; idx += W * kWave) {
            const int row = idx / COLS, c = idx % COLS;
            float v = 0.0f;
            if (row < m && c0 + c < p.cols) {
                float *xp = p.Xout + (size_t)(row0 + row) * p.ldx + c0 + c;
                v = *xp + s_tile[row * (COLS + 1) + c];
                *xp = v;
                // operand of the next RMSNorm-ed product: x (.) g
                put_act<P>(reinterpret_cast<T *>(p.An), act_plane(p.rr.cap, p.ldx),
                           act_idx<P>(row0 + row, c0 + c, p.ldx), v * p.gain[c0 + c]);
            }
            s_sq[idx] = v * v;
        }
        __syncthreads();
        if (tid < ROWS * NT) {
            const int row = tid / NT, j = tid % NT;
            if (row < m && (t0 + j) * 16 < p.cols) {
                float sum = 0.0f;
#pragma unroll
                for (int c = 0; c < 16; ++c) sum += s_sq[row * COLS + 16 * j + c];
                p.ssq_out[(size_t)(row0 + row) * p.T + t0 + j] = sum;
            }
        }
    } else if constexpr (EP == E_SWIGLU) {
        // Tiles come in (gate, up) pairs of the same 16 features.
        static_assert(NT % 2 == 0, "gate/up epilogue pairs a gate tile with an up tile");
        for (int idx = tid; idx < ROWS * COLS / 2; idx += W * kWave) {
            const int row = idx / (COLS / 2), f = idx % (COLS / 2), q = f >> 4, c = f & 15;
            if (row >= m || wg * COLS + 32 * q >= p.cols) continue;  // pair past the last column
            const float gt = s_tile[row * (COLS + 1) + 32 * q + c];
            const float up = s_tile[row * (COLS + 1) + 32 * q + 16 + c];
            put_act<P>(reinterpret_cast<T *>(p.H), act_plane(p.rr.cap, p.Fp),
                       act_idx<P>(row0 + row, wg * (COLS / 2) + f, p.Fp), silu(gt) * up);
        }
    } else if constexpr (EP == E_LOGITS) {
        // Plain fp32 output rows (the loss head's logits): Zout[row][col], col < V.
        const int c0 = t0 * 16;
        for (int idx = tid; idx < ROWS * COLS; idx += W * kWave) {
            const int row = idx / COLS, c = idx % COLS;
            if (row < m && c0 + c < p.V) p.Zout[(size_t)(row0 + row) * p.ldz + c0 + c] = s_tile[row * (COLS + 1) + c];
        }
    } else {  // E_ARGMAX
        // One wave per row: (max, lowest column) over this workgroup's columns < V.
        for (int row = w; row < ROWS; row += W) {
            if (row >= m) break;
            float bv = -INFINITY;
            int bi = 0x7fffffff;
            int nan = 0;
            for (int c = lane; c < COLS; c += kWave) {
                const int col = t0 * 16 + c;
                if (col < p.V) {
                    const float v = s_tile[row * (COLS + 1) + c];
                    if (p.dbg) p.dbg[(size_t)(row0 + row) * p.V + col] = v;
                    if (v != v) nan = 1;
                    else if (v > bv || (v == bv && col < bi)) { bv = v; bi = col; }
                }
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                const float ov = __shfl_xor(bv, off);
                const int oi = __shfl_xor(bi, off);
                nan |= __shfl_xor(nan, off);
                if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
            }
            if (lane == 0) {
                const size_t o = (size_t)(row0 + row) * ((p.cols + COLS - 1) / COLS) + wg;  // [row][column workgroup]
                p.pmax[o] = bv;
                p.pidx[o] = nan ? -1 : bi;
            }
        }
    }
}

// LDS floats of gemm_kernel's body
template <int NT, int RG, int W>
__host__ __device__ constexpr int tile_lds_floats() {
    return W * NT * 256 + 16 * RG * (16 * NT + 1) + kMaxRows;
}

// The body of gemm_kernel for column group wg, row tile p.rt0 + rt and K range z (E_LOGITS with
// p.kc > 0); smem holds tile_lds_floats<NT, RG, W>() floats.
template <Prec P, int NT, int RG, int EP, int D, int W, bool MT>
__device__ __forceinline__ void gemm_tile_body(GemmParams p, int wg, int rt, int z, float *smem, int row0_at = -1) {
    static_assert(W == 8, "the K split and its reduction tree are defined for 8 waves");
    constexpr bool ROWSCALE = EP != E_RESID && EP != E_LOGITS;  // the product follows an RMSNorm
    constexpr int ROWS = 16 * RG, COLS = 16 * NT;
    if constexpr (EP == E_LOGITS) {
        if (p.kc > 0) {  // split K: k-steps [z kc, min((z + 1) kc, Ks)), partial products to plane z
            const int ks0 = z * p.kc;
            p.W += (size_t)ks0 * (p.cols >> 4) * kTileBytes;
            p.A = reinterpret_cast<const uint8_t *>(p.A) + (size_t)ks0 * kWave * 16;  // 16-byte lane vectors
            p.Ks = min(p.kc, p.Ks - ks0);
            p.Zout += (size_t)z * p.zstride;
        }
    }
    // This workgroup's row tile: rows [row0, row0 + ROWS) of the iteration (within the row
    // capacity; row0_at, when given, places it); m of them are live. A launch of one row tile
    // (MT false) always has live rows, so nothing waits for the row count before the first loads;
    // with several row tiles (MT) a tile with no live row exits first.
    const int row0 = row0_at >= 0 ? row0_at : (p.rt0 + rt) * ROWS;
    request_together(p.W, p.A, p.ssq, p.Ks, p.cols, p.lda, p.rr.cap, p.T);
    const int m = p.rr.tab->R - row0;
    if constexpr (MT) {
        if (m <= 0) return;
    }
    const int rg0 = row0 >> 4;
    const int tid = threadIdx.x, lane = tid & 63;
    // wave index made explicitly wave-uniform, so k-step addresses live in scalar registers and
    // every load shares one per-lane offset
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = wg * NT;

    float *s_red = smem;                   // W waves x NT x 256 (also ROWS x COLS for E_RESID)
    float *s_tile = s_red + W * NT * 256;  // ROWS x (COLS + 1)
    float *s_inv = s_tile + ROWS * (COLS + 1);      // ROWS

    // Row factor inputs are requested before the weights (their latency overlaps the first
    // k-step's) and reduced after the main loop.
    f32x4 sq_pre[2];
    if constexpr (ROWSCALE) row_factor_preload<W>(p, row0, tid, sq_pre);

    // This wave's k-steps (nmy of them); the first D-1 are requested first.
    const int nmy = w < p.Ks ? (p.Ks - w + W - 1) / W : 0;
    auto step_of = [&](int q) { return min(w + q * W, p.Ks - 1); };
    Stage<P, NT, RG> ring[D];
#pragma unroll
    for (int j = 0; j < D - 1; ++j) gemm_load<P, NT, RG, MT>(ring[j], p, t0, rg0, step_of(j), lane);

    f32x4 acc[RG][NT];
#pragma unroll
    for (int r = 0; r < RG; ++r)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[r][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Software pipeline: a ring of D k-steps whose loads are in flight while the oldest one's
    // MFMAs run. The steady state is branch-free (exact wait counts); the drain issues no loads
    // past the end.
    if (nmy > 0) {
        // blocks of D steps whose prefetches (up to step b*D + 2D - 2) are all in range
        const int nfull = nmy >= 2 * D - 1 ? (nmy - (D - 1)) / D : 0;
        for (int bi = 0; bi < nfull; ++bi) {
#pragma unroll
            for (int j = 0; j < D; ++j) {
                // sched_barrier keeps the scheduler from sinking loads to their uses.
                gemm_load<P, NT, RG, MT>(ring[(j + D - 1) % D], p, t0, rg0, step_of(bi * D + j + D - 1), lane);
                __builtin_amdgcn_sched_barrier(0);
                gemm_compute(ring[j], acc);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        const int v0 = nfull * D;
#pragma unroll
        for (int j = 0; j < 2 * D - 1; ++j) {
            const int v = v0 + j;
            if (v < nmy) {
                if (v + D - 1 < nmy)
                    gemm_load<P, NT, RG, MT>(ring[(j + D - 1) % D], p, t0, rg0, step_of(v + D - 1), lane);
                gemm_compute(ring[j % D], acc);
            }
        }
    }

    if constexpr (ROWSCALE) row_factor_reduce<W, ROWS>(p, row0, tid, sq_pre, s_inv);

    // Sum of the 8 waves' partial tiles through LDS, one row group at a time, in the fixed tree
    // ((w0+w4)+(w2+w6))+((w1+w5)+(w3+w7)); then the RMSNorm row factor.
#pragma unroll
    for (int r = 0; r < RG; ++r) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
            *reinterpret_cast<f32x4 *>(s_red + ((size_t)(w * NT + j) * 64 + lane) * 4) = acc[r][j];
        __syncthreads();
        for (int e = tid; e < NT * 256; e += W * kWave) {
            float x[W];
#pragma unroll
            for (int q = 0; q < W; ++q) x[q] = s_red[(size_t)q * NT * 256 + e];
            float sum = ((x[0] + x[4]) + (x[2] + x[6])) + ((x[1] + x[5]) + (x[3] + x[7]));
            // element e = (tile j, lane l, register v); C layout: row 4*(l/16)+v, column l%16
            const int j = e >> 8, l = (e >> 2) & 63, v = e & 3;
            const int row = 16 * r + 4 * (l >> 4) + v;
            if constexpr (ROWSCALE) sum *= s_inv[row];
            s_tile[row * (COLS + 1) + 16 * j + (l & 15)] = sum;
        }
        __syncthreads();
    }

    gemm_epilogue<P, NT, RG, EP, W>(p, s_tile, s_red, row0, m, wg, tid, lane, w);
}

// gemm_kernel's body for row tile rt of a launch (rows from (p.rt0 + rt) 16 RG on) with only as
// many 16-row groups as the tile has live rows (at most RG). A row's sums do not depend on the
// row groups computed beside it, so every row keeps its values, and a tile of few rows (a
// shrinking block, the last tile of a batched iteration) streams the weights with fewer operand
// rows and MFMAs. A one-tile launch (MT false) reads the row count before its first loads (the
// host knows only the block size, not the rows each queued iteration will have); a launch of
// several tiles reads it anyway, to let dead tiles exit. smem holds tile_lds_floats<NT, RG, W>()
// floats.
template <Prec P, int NT, int RG, int EP, int D, int W, bool MT>
__device__ __forceinline__ void gemm_tile_body_live(const GemmParams &p, int wg, int rt, int z, float *smem) {
    if constexpr (RG > 1) {
        const int row0 = (p.rt0 + rt) * 16 * RG;
        const int m = p.rr.tab->R - row0;
        if (m <= 16) return gemm_tile_body<P, NT, 1, EP, D, W, MT>(p, wg, 0, z, smem, row0);
        if constexpr (RG > 2) {
            if (m <= 32) return gemm_tile_body<P, NT, 2, EP, D, W, MT>(p, wg, 0, z, smem, row0);
        }
        if constexpr (RG > 3) {
            if (m <= 48) return gemm_tile_body<P, NT, 3, EP, D, W, MT>(p, wg, 0, z, smem, row0);
        }
    }
    gemm_tile_body<P, NT, RG, EP, D, W, MT>(p, wg, rt, z, smem);
}

template <Prec P, int NT, int RG, int EP, int D, int W, bool MT>
__global__ __launch_bounds__(W * kWave) void gemm_kernel(GemmParams p) {
    extern __shared__ float smem[];
    gemm_tile_body_live<P, NT, RG, EP, D, W, MT>(p, blockIdx.x, blockIdx.y, blockIdx.z, smem);
}

// ------------------------------------------------------------------------------------------
// Prompt GEMM (prefill passes, bf16): Y[rows x N] = A[rows x K] * W^T over the same packed
// operands, for workgroup tiles of 16 RG rows x 16 NT columns. The 8 waves form a WM x (8 / WM)
// grid over the tile and each accumulates its sub-tile over every k-step in order (one MFMA per
// plane, hi then lo). The operands of a k-step (2 RG activation blocks and NT weight tiles of
// 1 KiB each) are loaded once per workgroup from global memory straight into LDS (LDS DMA), into a
// ring of NB buffers.
//
// What bounds it: the MFMAs and the clock. With random operands, 512 rows of the LLaMA-2-7B shape,
// gate/up takes 318k cycles, in which the MFMAs are busy 54% (69% of the 249k cycles in which a CU has
// waves; QKV and down alike, O 34%); LDS instructions take a fifth of a CU's cycles, without bank
// conflicts, and a CU pulls 35-45 GB/s of operands, where the former kernel's smaller tiles were held
// at 65-70. The clock is about 2.1 GHz then; with constant operands the same 302k cycles run at 2.5
// GHz (118 us for 145). Larger tiles move fewer bytes per MFMA, through LDS as from memory. Hence one
// workgroup per CU with a large tile (128 x 384 for gate/up: 160 KiB of LDS, 232 workgroups at 512
// rows), not several small ones. Each wave holds two sets of operand registers: while the MFMAs of a
// k-step run, the next k-step's operands are read from LDS between them, and the barrier of a k-step
// finds its operands already in registers. Four or five ring buffers measure alike, three too few.
// Measured at the LLaMA-2-7B shape, 512 rows, random operands, against the former kernel (64 x 256
// and 64 x 128 tiles, two or three workgroups per CU, the operands of a k-step read, waited for
// and then multiplied): gate/up 179 -> 150 us, QKV 119 -> 91, down (with its reduction) 102 -> 91,
// O 50 -> 50 (1.0-1.2 PFLOP/s of MFMA work). Prefetching a later k-step into L2 from the same waves
// was slower (194 us for gate/up): the prefetches wait in the same in-order queue.
//
// Ring: at k-step s a wave waits until its DMA blocks of k-step s + 1 have landed and its own LDS
// reads are complete, passes the barrier, issues k-step s + NB - 1 into the buffer of k-step s - 1
// and reads k-step s + 1. Every wave read buffer s - 1 before it computed k-step s - 1, so no
// reader is left when it is refilled. The barrier is issued without the compiler's LDS fence (which
// would wait for every outstanding DMA), with compiler-only fences so no LDS access moves across it.
//
// A row's reduction order depends only on K (and on the fixed K ranges of a split launch), never
// on the tile or the rows of a pass, so every prompt row gets the same values whatever the chunk
// size; the order differs from gemm_kernel's (which keeps eight k-step classes so decode rows are
// exact across row counts), so prompt rows always take this kernel. The RMSNorm row factors of
// prompt rows are computed once, by the kernel that writes the rows (embed_kernel,
// prompt_reduce_kernel), instead of by every workgroup from the sums of squares (3.5-4.5 us of
// each launch). Epilogues: through LDS into 16-byte vectors of the output's layout.
// ------------------------------------------------------------------------------------------
// floats per row of a wave's epilogue block (16-byte rows, spread over the banks)
template <int NT, int WM, int EP>
__host__ __device__ constexpr int prompt_row_floats() {
    return (EP == E_SWIGLU ? 8 : 16) * (NT / (kGemmWaves / WM)) + 4;
}
template <int NT, int RG, int WM, int EP, int NB, bool CLS = false>
__host__ __device__ constexpr int prompt_lds_bytes() {
    constexpr int stage = NB * (2 * RG + NT) * kTileBytes + (CLS && RG > 4 ? 16 * RG * 16 * NT * 4 : 0);
    constexpr int after = (kGemmWaves * (16 * RG / WM) * prompt_row_floats<NT, WM, EP>() + 16 * RG) * 4;
    return stage > after ? stage : after;
}

// CLS keeps gemm_kernel's reduction order instead: one accumulator per class of k-steps (k % 8), added
// in its tree ((0+4)+(2+6))+((1+5)+(3+7)) at the end. For the loss head's products, whose fp32 results
// leave the library as they are: a single chain is 3-6% further from 64 bits at the 7B head. Eight
// accumulators of a tile of more than 64 rows do not fit the registers, so it takes the even k-steps first, then
// the odd ones (four classes each; the weights are stored k-step by k-step, so the order of the
// visits costs nothing), with the even classes' sum held in LDS behind the ring meanwhile. (One
// accumulator and a fold after each class in turn: 3-4 us more a launch in register moves.)
template <int NT, int RG, int WM, int EP, int NB, bool CLS = false>
__global__ __launch_bounds__(kGemmWaves * kWave, 2) void gemm_prompt_kernel(GemmParams p) {
    constexpr Prec P = Prec::BF16;
    constexpr int W = kGemmWaves, WN = W / WM, RGW = RG / WM, NTW = NT / WN;
    constexpr int BLK = 2 * RG + NT, NLW = (BLK + W - 1) / W;  // 1 KiB blocks per k-step, DMA loads per wave
    static_assert(RG % WM == 0 && NT % WN == 0 && NB >= 4, "tile split, ring depth");
    static_assert(EP == E_QKV || EP == E_SWIGLU || EP == E_LOGITS, "the prompt products' epilogues");
    static_assert(EP != E_SWIGLU || NTW % 2 == 0, "a wave holds whole (gate, up) tile pairs");
    static_assert(EP != E_QKV || kWave % (16 * RGW) == 0, "QKV epilogue: a lane serves one row");
    constexpr bool ROWSCALE = EP != E_LOGITS;  // the product follows an RMSNorm
    constexpr int ROWS = 16 * RG, WROWS = 16 * RGW;
    // Workgroup L runs on XCD L % 8 (round-robin dispatch). Column group cg belongs to XCD cg % 8,
    // and each XCD takes its column groups in turn with their row tiles consecutively, so the row
    // tiles of a column group run together and read its weights once from HBM into that XCD's L2.
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int wg = (slot / p.row_tiles) * 8 + xcd, row0 = (slot % p.row_tiles) * ROWS;
    request_together(p.W, p.A, p.Ks, p.cols, p.lda, p.rr.cap, p.n_wg, p.rr.rows, p.rr.tab, p.sinv);
    const int m = p.rr.tab->R - row0;
    if (m <= 0 || wg >= p.n_wg) return;
    const int rg0 = row0 >> 4, t0 = wg * NT;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w / WN, wn = w % WN;
    const int wrow = wm * WROWS;     // the wave's first row of the tile
    const bool live = wrow < m;      // a wave whose rows are all past the pass only helps load
    // E_LOGITS with p.kc > 0: grid y takes k-steps [y kc, min((y + 1) kc, Ks)) and writes its
    // partial products to plane y
    int Ks = p.Ks, ks0 = 0;
    if constexpr (EP == E_LOGITS) {
        if (p.kc > 0) {
            ks0 = blockIdx.y * p.kc;
            Ks = min(p.kc, p.Ks - ks0);
            p.Zout += (size_t)blockIdx.y * p.zstride;
        }
    }
    extern __shared__ float smem[];
    u32x4 *s_stage = reinterpret_cast<u32x4 *>(smem);  // [NB][BLK][64] during the main loop

    // what the epilogue needs of the rows, requested before the main loop: the row factors (one
    // row per thread) and, for QKV, the position and slot of the lane's row
    float inv = 0.0f;
    if constexpr (ROWSCALE) {
        if (tid < ROWS) inv = p.sinv[row0 + tid];  // row0 + tid < row capacity (launcher)
    }
    const int erow = lane % WROWS;  // QKV: the lane's row of the wave's block
    int epos = 0, eslot = 0;
    if constexpr (EP == E_QKV) {
        if (wrow + erow < m) {
            const RowInfo ri = p.rr.rows[row0 + wrow + erow];
            epos = ri.pos;
            eslot = p.rr.tab->seq[ri.b];
        }
    }

    // This wave's blocks b = w + i W of every k-step: block b < 2 RG is activation plane b / RG,
    // row group b % RG; block 2 RG + j is weight tile t0 + j (clamped; its columns are never
    // written). Where the last round has no block for a wave, it loads the last block again into
    // its place, so every wave has the same number of loads in flight. A k-step advances an
    // activation block by 64 vectors and a weight block by one k-step of tiles.
    const int tiles = p.cols >> 4, ks_a = p.lda / PrecT<P>::KSTEP;
    const u32x4 *src[NLW];
    int adv[NLW], dst[NLW];
#pragma unroll
    for (int i = 0; i < NLW; ++i) {
        const int b = min(w + i * W, BLK - 1);
        dst[i] = b;
        if (b < 2 * RG) {
            const uint16_t *A = reinterpret_cast<const uint16_t *>(p.A) + (b / RG) * act_plane(p.rr.cap, p.lda);
            src[i] = reinterpret_cast<const u32x4 *>(A + (size_t)(rg0 + b % RG) * ks_a * kWave * 8) + lane;
            adv[i] = kWave;
        } else {
            src[i] = reinterpret_cast<const u32x4 *>(p.W + (size_t)min(t0 + b - 2 * RG, tiles - 1) * kTileBytes) + lane;
            adv[i] = tiles * kWave;
        }
        src[i] += (size_t)ks0 * adv[i];  // the first k-step of this workgroup's K range
    }
    // The next k-step of the order into ring buffer buf; past the last one a harmless reload of it.
    // With two passes the first one is padded to whole turns of the accumulators.
    constexpr int PASSES = CLS && RG > 4 ? 2 : 1, SETS = CLS ? 8 / PASSES : 1;
    int kn = 0;  // the next k-step to issue
    const int kodd = (((Ks + 1) >> 1) + SETS - 1) / SETS * SETS * 2;  // where the odd k-steps follow
    auto issue = [&](int buf) {
        const size_t ss = (size_t)min(kn, Ks - 1);
        u32x4 *bb = s_stage + (size_t)buf * BLK * kWave;
#pragma unroll
        for (int i = 0; i < NLW; ++i)
            __builtin_amdgcn_global_load_lds(static_cast<const void *>(src[i] + ss * adv[i]),
                                             (__attribute__((address_space(3))) void *)(bb + (size_t)dst[i] * kWave), 16,
                                             0, 0);
        kn += PASSES;
        if (PASSES == 2 && kn == kodd) kn = 1;
    };
#pragma unroll
    for (int q = 0; q < NB - 1; ++q) issue(q);

    f32x4 accs[SETS][RGW][NTW];
    auto clear = [&]() {
#pragma unroll
        for (int q = 0; q < SETS; ++q)
#pragma unroll
            for (int r = 0; r < RGW; ++r)
#pragma unroll
                for (int j = 0; j < NTW; ++j) accs[q][r][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    clear();
    u32x4 a[2][2][RGW], b[2][NTW];  // two sets: the k-step being computed, the next one
    auto read_operands = [&](auto set, int buf) {
        constexpr int st = decltype(set)::value;
        const u32x4 *bp = s_stage + (size_t)buf * BLK * kWave + lane;
#pragma unroll
        for (int j = 0; j < NTW; ++j) b[st][j] = bp[(2 * RG + wn * NTW + j) * kWave];
#pragma unroll
        for (int pl = 0; pl < 2; ++pl)
#pragma unroll
            for (int r = 0; r < RGW; ++r) a[st][pl][r] = bp[(pl * RG + wm * RGW + r) * kWave];
    };
    int rbuf = 1, ibuf = NB - 1;  // ring buffers of the next k-step and of the one NB - 1 ahead
    auto step = [&](auto set, auto which, bool add = true) {  // operand set, accumulator set
        constexpr int st = decltype(set)::value, ac = decltype(which)::value;
        wait_vm_lds<(NB - 3) * NLW>();  // this wave's blocks of the next k-step have landed
        barrier_no_fence();             // every wave's; buffer ibuf has no reader left
        issue(ibuf);
        if (live) {
            read_operands(std::integral_constant<int, st ^ 1>{}, rbuf);
            if (add) {
#pragma unroll
                for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                    for (int r = 0; r < RGW; ++r)
#pragma unroll
                        for (int j = 0; j < NTW; ++j) accs[ac][r][j] = mfma_kstep<P>(a[st][pl][r], b[st][j], accs[ac][r][j]);
            }
            // schedule: one LDS read after every few MFMAs
            constexpr int reads = 2 * RGW + NTW, mfmas = 2 * RGW * NTW, per = mfmas >= reads ? mfmas / reads : 1;
#pragma unroll
            for (int i = 0; i < reads; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // LDS read
                __builtin_amdgcn_sched_group_barrier(0x008, per, 0);  // MFMA
            }
            __builtin_amdgcn_sched_group_barrier(0x008, mfmas, 0);
        }
        rbuf = rbuf == NB - 1 ? 0 : rbuf + 1;
        ibuf = ibuf == NB - 1 ? 0 : ibuf + 1;
    };
    constexpr std::integral_constant<int, 0> set0{};
    constexpr std::integral_constant<int, 1> set1{};
    wait_vm<(NB - 2) * NLW>();  // this wave's blocks of k-step 0
    barrier_no_fence();
    if (live) read_operands(set0, 0);
    auto &acc = accs[0];
    if constexpr (CLS) {
        constexpr std::integral_constant<int, 2> set2{};
        constexpr std::integral_constant<int, 3> set3{};
        constexpr std::integral_constant<int, 4> set4{};
        constexpr std::integral_constant<int, 5> set5{};
        constexpr std::integral_constant<int, 6> set6{};
        constexpr std::integral_constant<int, 7> set7{};
        auto add = [&](int to, int from) {
#pragma unroll
            for (int r = 0; r < RGW; ++r)
#pragma unroll
                for (int j = 0; j < NTW; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) accs[to][r][j][e] += accs[from][r][j][e];
        };
        if constexpr (PASSES == 1) {
            int n = Ks;
            for (; n >= SETS; n -= SETS) {
                step(set0, set0);
                step(set1, set1);
                step(set0, set2);
                step(set1, set3);
                step(set0, set4);
                step(set1, set5);
                step(set0, set6);
                step(set1, set7);
            }
            if (n > 0) step(set0, set0);
            if (n > 1) step(set1, set1);
            if (n > 2) step(set0, set2);
            if (n > 3) step(set1, set3);
            if (n > 4) step(set0, set4);
            if (n > 5) step(set1, set5);
            if (n > 6) step(set0, set6);
            add(0, 4), add(2, 6), add(1, 5), add(3, 7);
            add(0, 2), add(1, 3);
            add(0, 1);
        } else {  // classes 0 2 4 6, then 1 3 5 7
            f32x4 *even = reinterpret_cast<f32x4 *>(s_stage + (size_t)NB * BLK * kWave) + tid;  // the lane's own places
            for (int ps = 0; ps < 2; ++ps) {
                const int n = (Ks + 1 - ps) >> 1;
                int g = 0;
                for (; g + SETS <= n; g += SETS) {
                    step(set0, set0);
                    step(set1, set1);
                    step(set0, set2);
                    step(set1, set3);
                }
                if (g < n) {  // the last turn, padded
                    step(set0, set0);
                    step(set1, set1, g + 1 < n);
                    step(set0, set2, g + 2 < n);
                    step(set1, set3, false);
                }
                add(0, 2), add(1, 3);
                add(0, 1);
                if (ps == 0) {
#pragma unroll
                    for (int r = 0; r < RGW; ++r)
#pragma unroll
                        for (int j = 0; j < NTW; ++j) even[(r * NTW + j) * W * kWave] = acc[r][j];
                    clear();
                }
            }
#pragma unroll
            for (int r = 0; r < RGW; ++r)
#pragma unroll
                for (int j = 0; j < NTW; ++j) {
                    const f32x4 x = even[(r * NTW + j) * W * kWave];
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[r][j][e] = x[e] + acc[r][j][e];
                }
        }
    } else {
        int s = 0;
        for (; s + 2 <= Ks; s += 2) {
            step(set0, set0);
            step(set1, set0);
        }
        if (s < Ks) step(set0, set0);
    }
    wait_vm<0>();  // the trailing reloads have landed before the buffers are reused
    __syncthreads();

    // The wave's outputs into its LDS block (C layout of a 16 x 16 tile: lane l, register v -> row
    // 4 (l / 16) + v, column l % 16), then out as vectors.
    constexpr int LDR = prompt_row_floats<NT, WM, EP>();
    float *s_w = smem + (size_t)w * WROWS * LDR;
    float *s_inv = smem + (size_t)W * WROWS * LDR;
    if constexpr (ROWSCALE) {
        if (tid < ROWS) s_inv[tid] = inv;
        __syncthreads();
    }
    if (!live) return;
    const int c16 = lane & 15, r4 = 4 * (lane >> 4);
#pragma unroll
    for (int r = 0; r < RGW; ++r) {
        f32x4 iv = f32x4{1.f, 1.f, 1.f, 1.f};
        if constexpr (ROWSCALE) iv = *reinterpret_cast<const f32x4 *>(s_inv + wrow + 16 * r + r4);
        if constexpr (EP == E_SWIGLU) {
#pragma unroll
            for (int j = 0; j < NTW; j += 2)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float g = acc[r][j][v] * iv[v], u = acc[r][j + 1][v] * iv[v];
                    s_w[(16 * r + r4 + v) * LDR + 8 * j + c16] = silu(g) * u;
                }
        } else {
#pragma unroll
            for (int j = 0; j < NTW; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float x = acc[r][j][v];
                    if constexpr (ROWSCALE) x *= iv[v];
                    s_w[(16 * r + r4 + v) * LDR + 16 * j + c16] = x;
                }
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // the wave reads back its own block only
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if constexpr (EP == E_SWIGLU) {
        uint16_t *H = reinterpret_cast<uint16_t *>(p.H);
#pragma unroll 2
        for (int i = lane; i < WROWS * NTW; i += kWave) {  // NTW vectors of 8 features per row
            const int row = i % WROWS, q = i / WROWS;
            const int t = t0 + wn * NTW + (q & ~1);  // the gate tile of the pair
            if (wrow + row >= m || t >= tiles) continue;
            alignas(16) float x[8];
            *reinterpret_cast<f32x4 *>(x) = *reinterpret_cast<const f32x4 *>(s_w + row * LDR + 8 * q);
            *reinterpret_cast<f32x4 *>(x + 4) = *reinterpret_cast<const f32x4 *>(s_w + row * LDR + 8 * q + 4);
            put_act8(H, act_plane(p.rr.cap, p.Fp), act_idx<P>(row0 + wrow + row, t * 8 + 8 * (q & 1), p.Fp), x);
        }
    } else if constexpr (EP == E_QKV) {
        // One tile of the lane's row at a time: 8 dims of a head and their 8 rotate-half partners.
        const int hd = p.hd, d = p.d, h2 = hd >> 1;
        if (wrow + erow >= m) return;
        const size_t kvs = (size_t)eslot * p.kv_seq;
        for (int j = lane / WROWS; j < NTW; j += kWave / WROWS) {
            const int R0 = (t0 + wn * NTW + j) * 16;
            if (R0 >= p.cols) break;
            const int sec = R0 / d, within = R0 % d, head = within / hd, dim = (within % hd) >> 1;
            const size_t kvo = kvs + (size_t)head * p.ctx_alloc * hd;
            alignas(16) float x[16];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<f32x4 *>(x + 4 * q) = *reinterpret_cast<const f32x4 *>(s_w + erow * LDR + 16 * j + 4 * q);
            if (sec < 2) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const f32x4 c = *reinterpret_cast<const f32x4 *>(p.rcos + (size_t)epos * h2 + dim + 4 * q);
                    const f32x4 sn = *reinterpret_cast<const f32x4 *>(p.rsin + (size_t)epos * h2 + dim + 4 * q);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float u = x[4 * q + e], y = x[8 + 4 * q + e];
                        x[4 * q + e] = u * c[e] - y * sn[e];
                        x[8 + 4 * q + e] = y * c[e] + u * sn[e];
                    }
                }
            }
            if (sec == 0) {
                uint16_t *Q = reinterpret_cast<uint16_t *>(p.Q);
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    put_act8(Q, act_plane(p.rr.cap, d), act_idx<P>(row0 + wrow + erow, head * hd + h * h2 + dim, d), x + 8 * h);
            } else {  // cached keys and values are rounded to the cache dtype
                alignas(16) uint16_t y[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) y[e] = f2bf(x[e]);
                if (sec == 1) {
                    uint16_t *Kc = reinterpret_cast<uint16_t *>(p.Kc) + kvo;
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        *reinterpret_cast<u32x4 *>(Kc + kcache_idx<P>(epos, h * h2 + dim, hd)) =
                            *reinterpret_cast<const u32x4 *>(y + 8 * h);
                } else {
                    uint16_t *Vt = reinterpret_cast<uint16_t *>(p.Vt) + kvo;
#pragma unroll
                    for (int e = 0; e < 16; ++e) Vt[vcache_idx<P>(epos, (e >> 3) * h2 + dim + (e & 7), hd)] = y[e];
                }
            }
        }
    } else {  // E_LOGITS: fp32 rows
        constexpr int VPR = 4 * NTW;
#pragma unroll 4
        for (int i = lane; i < WROWS * VPR; i += kWave) {
            const int row = i / VPR, q = i % VPR;
            const int c = (t0 + wn * NTW) * 16 + 4 * q;
            if (wrow + row < m && c < p.cols)
                *reinterpret_cast<f32x4 *>(p.Zout + (size_t)(row0 + wrow + row) * p.ldz + c) =
                    *reinterpret_cast<const f32x4 *>(s_w + row * LDR + 4 * q);
        }
    }
}

// ------------------------------------------------------------------------------------------
// Row-tiled decode GEMM (iterations of more than 64 rows, bf16): workgroup tiles of 64 rows x
// 16 NT columns with the operand blocks brought into LDS by DMA (as gemm_prompt_kernel, NB
// buffers, NB - 1 k-steps in flight) and gemm_kernel's reduction order, so that every row gets
// the bits a one-tile iteration gives it (batched, AR and Jacobi decoding stay bit-identical):
// k-step k is accumulated into the set of its class k % 8 (from zero, the hi then the lo MFMA, in
// increasing k, as wave k % 8 of gemm_kernel accumulates it), and the eight class sums are folded
// at the end in gemm_kernel's tree ((x0 + x4) + (x2 + x6)) + ((x1 + x5) + (x3 + x7)). The RMSNorm
// row factor and the epilogues are gemm_kernel's. With p.kc > 0 (E_LOGITS) grid z splits K into
// ranges of kc k-steps, the classes of a range counted from its first k-step, as gemm_kernel
// splits it.
// ------------------------------------------------------------------------------------------
// tiles (16 columns) per workgroup and ring depth of the row-tiled products (measured at the
// LLaMA-2-7B shape, 96 to 512 rows; QKV and O stay faster on gemm_kernel)
constexpr int kRowsNtGateUp = 12, kRowsNbGateUp = 4;
constexpr int kRowsNtDown = 8, kRowsNbDown = 4;

template <int NT, int EP, int NB>
__host__ __device__ constexpr int rows_lds_floats() {
    constexpr int RG = 4, ROWS = 16 * RG, COLS = 16 * NT, BLK = 2 * RG + NT;
    constexpr int stage = NB * BLK * kWave * 4;
    constexpr int after = (EP == E_RESID ? ROWS * COLS : 0) + ROWS * (COLS + 1);
    return (stage > after ? stage : after) + ROWS;
}

// The row-tiled product of one tile of 16 RGT live rows (row0 on, m of them live) over a WM x
// (8 / WM) wave grid: eight class sums per output folded in gemm_kernel's tree, its row factor
// and epilogue. smem holds rows_lds_floats<NT, EP, NB>() floats (the launch's 64-row tile).
template <int RGT, int WM, int NT, int EP, int NB>
__device__ __forceinline__ void rows_tile_body(const GemmParams &p, int wg, int row0, int m, float *smem) {
    constexpr Prec P = Prec::BF16;
    constexpr int W = kGemmWaves, WN = W / WM, RGW = RGT / WM, NTW = NT / WN;
    constexpr int BLK = 2 * RGT + NT;
    static_assert(RGT % WM == 0 && NT % WN == 0 && NB >= 3, "tile split, ring depth");
    constexpr bool ROWSCALE = EP != E_RESID && EP != E_LOGITS;
    constexpr int ROWS = 16 * RGT, COLS = 16 * NT;
    const int rg0 = row0 >> 4, t0 = wg * NT;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w / WN, wn = w % WN;
    const int Ks = p.Ks;

    u32x4 *s_stage = reinterpret_cast<u32x4 *>(smem);  // [NB][BLK][64] during the main loop
    float *s_red = smem;
    float *s_tile = smem + (EP == E_RESID ? ROWS * COLS : 0);
    float *s_inv = smem + rows_lds_floats<NT, EP, NB>() - kMaxRows;

    f32x4 sq_pre[2];
    if constexpr (ROWSCALE) row_factor_preload<W>(p, row0, tid, sq_pre);

    // DMA blocks of a k-step: block b < 2 RGT is activation plane b / RGT, row group b % RGT;
    // block 2 RGT + j is weight tile t0 + j (clamped; its columns are never written). Wave w
    // issues blocks w, w + W, ... (NLW of them; where the last round has no block for a wave, it
    // loads the last block again into its place), so every wave has the same number of loads in
    // flight.
    constexpr int NLW = (BLK + W - 1) / W;
    const int tiles = p.cols >> 4, ks_a = p.lda / PrecT<P>::KSTEP;
    const u32x4 *src[NLW];
    int adv[NLW], dst[NLW];
#pragma unroll
    for (int i = 0; i < NLW; ++i) {
        const int b = min(w + i * W, BLK - 1);
        dst[i] = b;
        if (b < 2 * RGT) {
            const uint16_t *A = reinterpret_cast<const uint16_t *>(p.A) + (b / RGT) * act_plane(p.rr.cap, p.lda);
            src[i] = reinterpret_cast<const u32x4 *>(A + (size_t)(rg0 + b % RGT) * ks_a * kWave * 8) + lane;
            adv[i] = kWave;
        } else {
            src[i] = reinterpret_cast<const u32x4 *>(p.W + (size_t)min(t0 + b - 2 * RGT, tiles - 1) * kTileBytes) + lane;
            adv[i] = tiles * kWave;
        }
    }
    auto issue = [&](int s, int buf) {  // k-step s (< Ks) into ring buffer buf
        u32x4 *bb = s_stage + (size_t)buf * BLK * kWave;
#pragma unroll
        for (int i = 0; i < NLW; ++i)
            __builtin_amdgcn_global_load_lds(static_cast<const void *>(src[i] + (size_t)s * adv[i]),
                                             (__attribute__((address_space(3))) void *)(bb + (size_t)dst[i] * kWave),
                                             16, 0, 0);
    };
    // one accumulator set per class: k-step k goes to set k % 8, the k-steps in increasing order
    f32x4 acc[8][RGW][NTW];
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int r = 0; r < RGW; ++r)
#pragma unroll
            for (int j = 0; j < NTW; ++j) acc[c][r][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // past the last k-step the ring reloads k-step Ks - 1 (harmless, never computed)
#pragma unroll
    for (int q = 0; q < NB - 1; ++q) issue(min(q, Ks - 1), q);
    int buf = 0;  // ring buffer of the k-step being computed
    for (int k0 = 0; k0 < Ks; k0 += 8) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int k = k0 + c;
            if (k < Ks) {  // uniform over the workgroup
                wait_vm<(NB - 2) * NLW>();  // this wave's blocks of k-step k have landed
                barrier_no_fence();         // every wave's; the buffer refilled next has no reader left
                issue(min(k + NB - 1, Ks - 1), buf == 0 ? NB - 1 : buf - 1);
                const u32x4 *bp = s_stage + (size_t)buf * BLK * kWave + lane;
                u32x4 a[2][RGW], b[NTW];
#pragma unroll
                for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                    for (int r = 0; r < RGW; ++r) a[pl][r] = bp[(pl * RGT + wm * RGW + r) * kWave];
#pragma unroll
                for (int j = 0; j < NTW; ++j) b[j] = bp[(2 * RGT + wn * NTW + j) * kWave];
#pragma unroll
                for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                    for (int r = 0; r < RGW; ++r)
#pragma unroll
                        for (int j = 0; j < NTW; ++j) acc[c][r][j] = mfma_kstep<P>(a[pl][r], b[j], acc[c][r][j]);
                buf = buf == NB - 1 ? 0 : buf + 1;
            }
        }
    }
    wait_vm<0>();  // the trailing reloads have landed before the buffers are reused
    __syncthreads();

    if constexpr (ROWSCALE) row_factor_reduce<W, ROWS>(p, row0, tid, sq_pre, s_inv);
    __syncthreads();
    // gemm_kernel's tree over the class sums, then its row factor
#pragma unroll
    for (int r = 0; r < RGW; ++r)
#pragma unroll
        for (int j = 0; j < NTW; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * (wm * RGW + r) + 4 * (lane >> 4) + v;
                float x = ((acc[0][r][j][v] + acc[4][r][j][v]) + (acc[2][r][j][v] + acc[6][r][j][v])) +
                          ((acc[1][r][j][v] + acc[5][r][j][v]) + (acc[3][r][j][v] + acc[7][r][j][v]));
                if constexpr (ROWSCALE) x *= s_inv[row];
                s_tile[row * (COLS + 1) + 16 * (wn * NTW + j) + (lane & 15)] = x;
            }
    __syncthreads();
    gemm_epilogue<P, NT, RGT, EP, W>(p, s_tile, s_red, row0, m, wg, tid, lane, w);
}

// An iteration of at most 64 rows (one row tile; the row count is known only on the device) takes
// gemm_kernel's body with NT_T tiles per workgroup and D_T k-steps in flight instead: its column
// groups are narrower, so more workgroups share the work (one row tile of the row-tiled kernel
// would occupy fewer than half the CUs). The last live tile of a longer iteration runs only its
// live 16-row groups.
template <int NT, int EP, int NB, int NT_T, int D_T>
__global__ __launch_bounds__(kGemmWaves * kWave) void gemm_rows_kernel(GemmParams p) {
    constexpr Prec P = Prec::BF16;
    constexpr int RG = 4, W = kGemmWaves;
    constexpr int ROWS = 16 * RG;
    extern __shared__ float smem[];
    request_together(p.rr.tab, p.cols, p.rt0);
    if (p.rr.tab->R - p.rt0 * ROWS <= ROWS) {
        const int nwt = (p.cols + 16 * NT_T - 1) / (16 * NT_T);
        if ((int)blockIdx.x < nwt) gemm_tile_body_live<P, NT_T, RG, EP, D_T, W, true>(p, blockIdx.x, 0, blockIdx.z, smem);
        return;
    }
    if constexpr (EP == E_LOGITS) {
        if (p.kc > 0) {  // split K as gemm_kernel does
            const int ks0 = blockIdx.z * p.kc;
            p.W += (size_t)ks0 * (p.cols >> 4) * kTileBytes;
            p.A = reinterpret_cast<const uint8_t *>(p.A) + (size_t)ks0 * kWave * 16;
            p.Ks = min(p.kc, p.Ks - ks0);
            p.Zout += (size_t)blockIdx.z * p.zstride;
        }
    }
    // Column groups on XCDs in turn, the live row tiles of a column group consecutive on one XCD
    // (its L2 serves the weight tiles to all of them). The launch covers its largest row count; the
    // live row tiles (from the device row table) take the first workgroups of each XCD, so the
    // workgroups past them, which exit at once, are dispatched last.
    request_together(p.W, p.A, p.ssq, p.Ks, p.cols, p.lda, p.rr.cap, p.T, p.n_wg, p.row_tiles);
    const int live = min(p.row_tiles, (p.rr.tab->R - p.rt0 * ROWS + ROWS - 1) / ROWS);
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int wg = (slot / live) * 8 + xcd, row0 = (p.rt0 + slot % live) * ROWS;
    if (wg >= p.n_wg) return;
    const int m = p.rr.tab->R - row0;
    // 16-row groups of this tile with live rows (every row's values are the same whatever the
    // tile's row groups and wave grid); one or three groups take a one-row wave grid, which needs
    // NT a multiple of the 8 waves
    if constexpr (NT % W == 0) {
        if (m <= 16) return rows_tile_body<1, 1, NT, EP, NB>(p, wg, row0, m, smem);
        if (m <= 32) return rows_tile_body<2, 2, NT, EP, NB>(p, wg, row0, m, smem);
        if (m <= 48) return rows_tile_body<3, 1, NT, EP, NB>(p, wg, row0, m, smem);
    } else {
        if (m <= 32) return rows_tile_body<2, 2, NT, EP, NB>(p, wg, row0, m, smem);
    }
    rows_tile_body<4, 2, NT, EP, NB>(p, wg, row0, m, smem);
}

template <int NT, int EP, int NB, int NT_T, int D_T>
static hipError_t launch_rows_t(const GemmParams &p, int row_tiles, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    constexpr int COLS = 16 * NT;
    constexpr int lds_rows = rows_lds_floats<NT, EP, NB>(), lds_tile = tile_lds_floats<NT_T, 4, kGemmWaves>();
    const size_t lds = (size_t)(lds_rows > lds_tile ? lds_rows : lds_tile) * sizeof(float);
    if (row_tiles < 1 || (p.rt0 + row_tiles) * 64 > p.rr.cap || p.lda % 32 != 0 || p.cols % 16 != 0)
        return hipErrorInvalidValue;
    if (EP != E_LOGITS && p.kc != 0) return hipErrorInvalidValue;
    GemmParams q = p;
    q.n_wg = (p.cols + COLS - 1) / COLS;
    q.row_tiles = row_tiles;
    const int splits = EP == E_LOGITS && p.kc > 0 ? (p.Ks + p.kc - 1) / p.kc : 1;
    const int n_tile = (p.cols + 16 * NT_T - 1) / (16 * NT_T);  // column groups of the one-tile body
    const dim3 grid((unsigned)std::max((q.n_wg + 7) / 8 * 8 * row_tiles, n_tile), 1, (unsigned)splits);
    auto kern = gemm_rows_kernel<NT, EP, NB, NT_T, D_T>;
    if (e0 || e1)
        hipExtLaunchKernelGGL(kern, grid, dim3(kGemmWaves * kWave), lds, s, e0, e1, 0, q);
    else
        hipLaunchKernelGGL(kern, grid, dim3(kGemmWaves * kWave), lds, s, q);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Class-pair K split of the decode GEMM (bf16, iterations of more than 64 rows). gemm_kernel's
// tree ((x0 + x4) + (x2 + x6)) + ((x1 + x5) + (x3 + x7)) over the eight k-step class sums equals
// (t0 + t2) + (t1 + t3) with t_c = x_c + x_(c+4). Grid z = c in {0, 1, 2, 3}: a workgroup walks
// the k-steps k = c (mod 4) in increasing order and accumulates those with k = c (mod 8) into one
// set and those with k = c + 4 (mod 8) into another (from zero, the hi then the lo MFMA, as wave
// k % 8 of gemm_kernel accumulates them), then writes t_c of its 16 RGT x 16 NT tile, fp32, to
// plane c of p.spart; gemm_split_reduce_kernel forms (t0 + t2) + (t1 + t3), applies the RMSNorm
// row factor and runs gemm_kernel's epilogue. Every row therefore gets the bits of a one-tile
// iteration. Two accumulator sets instead of eight allow workgroup tiles four times larger (each
// k-step's operand rows and weight tiles, brought into LDS by DMA through a ring of NB buffers,
// serve more outputs), and the four K quarters are four times finer units of work. An iteration
// whose live rows fit one 64-row tile (known only on the device) takes gemm_kernel's body with
// NT_T tiles per workgroup and D_T k-steps in flight inside the split launch, and the reduction
// launch then has nothing to do.
//
// p.spart, plane c: [row group of 16 rows][16-column tile][lane][4] fp32 in the MFMA's C layout
// (lane l, register v: row 4 (l / 16) + v, column l % 16 of the tile), row capacity x p.cols
// floats per plane.
// ------------------------------------------------------------------------------------------
// 16-column tiles per workgroup and ring depth of the split products (64-row tiles; measured at
// the LLaMA-2-7B shape, 160 and 512 rows: gate/up 74.6 / 195 us, QKV 45.0 / 100 us before the
// reduction; O is no faster than gemm_kernel once its reduction is added)
constexpr int kSplitNtQkv = 16, kSplitNbQkv = 3, kSplitNtGateUp = 16, kSplitNbGateUp = 3;
constexpr int kSplitNtLm = 16, kSplitNbLm = 3;

template <int RGT, int NT, int NB>
__host__ __device__ constexpr int split_lds_floats() {
    return NB * (2 * RGT + NT) * kWave * 4;
}

// The class-pair product of one tile of 16 RGT live rows (row0 on): the k-steps c, c + 4, ... into
// two accumulator sets over a WM x (8 / WM) wave grid, t_c written to plane c of p.spart.
// smem holds split_lds_floats<4, NT, NB>() floats (the launch's 64-row tile).
template <int RGT, int WM, int NT, int NB>
__device__ __forceinline__ void split_tile_body(const GemmParams &p, int c, int wg, int row0, float *smem) {
    constexpr Prec P = Prec::BF16;
    constexpr int W = kGemmWaves, WN = W / WM, RGW = RGT / WM, NTW = NT / WN;
    constexpr int BLK = 2 * RGT + NT, NLW = (BLK + W - 1) / W;
    static_assert(RGT % WM == 0 && NT % WN == 0 && NB >= 3, "tile split, ring depth");
    const int rg0 = row0 >> 4, t0 = wg * NT;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w / WN, wn = w % WN;
    const int nq = (p.Ks - c + 3) >> 2;  // k-steps c, c + 4, ... below Ks (the launcher has Ks >= 4)
    const int last = c + 4 * (nq - 1);

    u32x4 *s_stage = reinterpret_cast<u32x4 *>(smem);  // [NB][BLK][64]
    // DMA blocks of a k-step: block b < 2 RGT is activation plane b / RGT, row group b % RGT; block
    // 2 RGT + j is weight tile t0 + j (clamped; its columns are never written). Wave w issues blocks
    // w, w + W, ... (NLW of them; where the last round has no block for a wave, it loads the last
    // block again into its place), so every wave has the same number of loads in flight.
    const int tiles = p.cols >> 4, ks_a = p.lda / PrecT<P>::KSTEP;
    const u32x4 *src[NLW];
    int adv[NLW], dst[NLW];
#pragma unroll
    for (int i = 0; i < NLW; ++i) {
        const int b = min(w + i * W, BLK - 1);
        dst[i] = b;
        if (b < 2 * RGT) {
            const uint16_t *A = reinterpret_cast<const uint16_t *>(p.A) + (b / RGT) * act_plane(p.rr.cap, p.lda);
            src[i] = reinterpret_cast<const u32x4 *>(A + (size_t)(rg0 + b % RGT) * ks_a * kWave * 8) + lane;
            adv[i] = kWave;
        } else {
            src[i] = reinterpret_cast<const u32x4 *>(p.W + (size_t)min(t0 + b - 2 * RGT, tiles - 1) * kTileBytes) + lane;
            adv[i] = tiles * kWave;
        }
    }
    auto issue = [&](int k, int buf) {  // k-step k (< Ks) into ring buffer buf
        u32x4 *bb = s_stage + (size_t)buf * BLK * kWave;
#pragma unroll
        for (int i = 0; i < NLW; ++i)
            __builtin_amdgcn_global_load_lds(static_cast<const void *>(src[i] + (size_t)k * adv[i]),
                                             (__attribute__((address_space(3))) void *)(bb + (size_t)dst[i] * kWave),
                                             16, 0, 0);
    };
    f32x4 acc[2][RGW][NTW];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < RGW; ++r)
#pragma unroll
            for (int j = 0; j < NTW; ++j) acc[h][r][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // past the last k-step the ring reloads the last one (harmless, never computed)
#pragma unroll
    for (int q = 0; q < NB - 1; ++q) issue(min(c + 4 * q, last), q);
    int buf = 0;  // ring buffer of the k-step being computed
    for (int q0 = 0; q0 < nq; q0 += 2) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {  // k-step c + 4 (q0 + h): class c for h = 0, c + 4 for h = 1
            const int q = q0 + h;
            if (q < nq) {  // uniform over the workgroup
                wait_vm<(NB - 2) * NLW>();  // this wave's blocks of the k-step have landed
                barrier_no_fence();         // every wave's; the buffer refilled next has no reader left
                issue(min(c + 4 * (q + NB - 1), last), buf == 0 ? NB - 1 : buf - 1);
                const u32x4 *bp = s_stage + (size_t)buf * BLK * kWave + lane;
                u32x4 a[2][RGW], b[NTW];
#pragma unroll
                for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                    for (int r = 0; r < RGW; ++r) a[pl][r] = bp[(pl * RGT + wm * RGW + r) * kWave];
#pragma unroll
                for (int j = 0; j < NTW; ++j) b[j] = bp[(2 * RGT + wn * NTW + j) * kWave];
#pragma unroll
                for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                    for (int r = 0; r < RGW; ++r)
#pragma unroll
                        for (int j = 0; j < NTW; ++j) acc[h][r][j] = mfma_kstep<P>(a[pl][r], b[j], acc[h][r][j]);
                buf = buf == NB - 1 ? 0 : buf + 1;
            }
        }
    }
    wait_vm<0>();  // the trailing reloads have landed before the workgroup ends

    float *Z = p.spart + (size_t)c * p.rr.cap * p.cols;
#pragma unroll
    for (int r = 0; r < RGW; ++r)
#pragma unroll
        for (int j = 0; j < NTW; ++j) {
            const int t = t0 + wn * NTW + j;
            if (t < tiles) {
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[0][r][j][e] + acc[1][r][j][e];
                *reinterpret_cast<f32x4 *>(Z + (((size_t)(rg0 + wm * RGW + r) * tiles + t) * kWave + lane) * 4) = v;
            }
        }
}

// The split product of a launch of several 64-row tiles, whatever the rows the iteration turns
// out to have (known only on the device): one that fits one tile takes the same path (the same
// values as gemm_kernel's). The kernel keeps to 128 registers (at least four waves per SIMD), so
// two workgroups share a CU.
template <int NT, int NB, int EP>
__global__ __launch_bounds__(kGemmWaves * kWave, 4) void gemm_split_kernel(GemmParams p) {
    constexpr int W = kGemmWaves;
    constexpr int ROWS = kMaxRows;
    extern __shared__ float smem[];
    // Column groups on XCDs in turn, the live row tiles of a column group consecutive on one XCD;
    // the launch covers its largest row count, the live row tiles take the first workgroups of
    // each XCD and the others exit at once.
    constexpr bool ROWSCALE = EP != E_RESID && EP != E_LOGITS;
    request_together(p.rr.tab, p.cols, p.rt0, p.W, p.A, p.Ks, p.lda, p.rr.cap, p.n_wg, p.row_tiles, p.spart, p.ssq,
                     p.T);
    const int R = p.rr.tab->R;
    if (R - p.rt0 * ROWS <= 0) return;
    const int live = min(p.row_tiles, (R - p.rt0 * ROWS + ROWS - 1) / ROWS);
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    // XCD x takes class pair x % 4 and every other column group from x / 4
    const int c = xcd & 3, wg = (slot / live) * 2 + (xcd >> 2);
    const int row0 = (p.rt0 + slot % live) * ROWS;
    if (wg >= p.n_wg) return;
    const int tid = threadIdx.x;
    // one workgroup per row tile also computes the tile's RMSNorm row factors for the reduction
    const bool factors = ROWSCALE && wg == 0 && c == 0;
    f32x4 sq_pre[2];
    if (factors) row_factor_preload<W>(p, row0, tid, sq_pre);

    // The last live tile runs only its live 16-row groups (rows past the iteration's rows have
    // no partials; the reduction writes nothing for them). Every row's t_c is the same whatever
    // the tile's row groups and wave grid; one or three groups take a one-row wave grid, which
    // needs NT a multiple of the 8 waves.
    const int mt = R - row0;
    if constexpr (NT % W == 0) {
        if (mt <= 16)
            split_tile_body<1, 1, NT, NB>(p, c, wg, row0, smem);
        else if (mt <= 32)
            split_tile_body<2, 2, NT, NB>(p, c, wg, row0, smem);
        else if (mt <= 48)
            split_tile_body<3, 1, NT, NB>(p, c, wg, row0, smem);
        else
            split_tile_body<4, 2, NT, NB>(p, c, wg, row0, smem);
    } else {
        if (mt <= 32)
            split_tile_body<2, 2, NT, NB>(p, c, wg, row0, smem);
        else
            split_tile_body<4, 2, NT, NB>(p, c, wg, row0, smem);
    }

    if (factors) {  // uniform over the workgroup
        __syncthreads();  // every wave is past its last read of the ring
        float *s_inv = smem;
        row_factor_reduce<W, ROWS>(p, row0, tid, sq_pre, s_inv);
        __syncthreads();
        if (tid < ROWS) p.sinv[row0 + tid] = s_inv[tid];
    }
}

// (t0 + t2) + (t1 + t3) of the class-pair partials for a 64-row tile x 16 NT columns, the RMSNorm
// row factor (computed once per row tile by the split launch) and gemm_kernel's epilogue. Grid: column groups x row tiles (from p.rt0); row tiles
// past the iteration's rows exit.
template <int NT, int EP>
__host__ __device__ constexpr int split_reduce_lds_floats() {
    constexpr int ROWS = kMaxRows, COLS = 16 * NT;
    return (EP == E_RESID ? ROWS * COLS : 0) + ROWS * (COLS + 1) + ROWS;
}

template <int NT, int EP>
__global__ __launch_bounds__(kGemmWaves * kWave) void gemm_split_reduce_kernel(GemmParams p) {
    constexpr Prec P = Prec::BF16;
    constexpr int W = kGemmWaves, RG = kMaxRows / 16, ROWS = kMaxRows, COLS = 16 * NT;
    constexpr int NV = RG * NT * kWave / (W * kWave);  // 16-byte vectors per thread and plane
    static_assert((RG * NT) % W == 0, "every thread takes the same number of vectors");
    constexpr bool ROWSCALE = EP != E_RESID && EP != E_LOGITS;
    extern __shared__ float smem[];
    const int wg = blockIdx.x, row0 = (p.rt0 + blockIdx.y) * ROWS;
    request_together(p.rr.tab, p.spart, p.cols, p.rr.cap, p.sinv, p.rt0);
    const int m = p.rr.tab->R - row0;
    if (m <= 0) return;  // a row tile past the iteration's rows
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    float *s_red = smem;                                       // epilogue scratch (E_RESID)
    float *s_tile = smem + (EP == E_RESID ? ROWS * COLS : 0);  // ROWS x (COLS + 1)
    float *s_inv = s_tile + ROWS * (COLS + 1);                 // ROWS
    const int tiles = p.cols >> 4, t0 = wg * NT, rg0 = row0 >> 4;
    const size_t plane = (size_t)p.rr.cap * p.cols;
    // vector u = tid + i W 64: row group (u / 64) / NT, tile (u / 64) % NT, lane u % 64; row
    // groups past the iteration's rows (the split launch wrote no partials there; their rows are
    // not written out) load nothing
    f32x4 z[NV][4];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int u = tid + i * W * kWave, blk = u >> 6;
        const int r = blk / NT, t = min(t0 + blk % NT, tiles - 1);
        const float *src = p.spart + (((size_t)(rg0 + r) * tiles + t) * kWave + (u & 63)) * 4;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            z[i][c] = 16 * r < m ? *reinterpret_cast<const f32x4 *>(src + c * plane) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if constexpr (ROWSCALE) {  // the row factors the split launch computed (row_factor_reduce's values)
        if (tid < ROWS) s_inv[tid] = p.sinv[row0 + tid];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int u = tid + i * W * kWave, blk = u >> 6, l = u & 63;
        const int r = blk / NT, j = blk % NT;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = 16 * r + 4 * (l >> 4) + v;
            float x = (z[i][0][v] + z[i][2][v]) + (z[i][1][v] + z[i][3][v]);
            if constexpr (ROWSCALE) x *= s_inv[row];
            s_tile[row * (COLS + 1) + 16 * j + (l & 15)] = x;
        }
    }
    __syncthreads();
    gemm_epilogue<P, NT, RG, EP, W>(p, s_tile, s_red, row0, m, wg, tid, lane, w);
}

// The product through the class-pair split: gemm_split_kernel over row_tiles tiles of 64 rows (from
// row tile p.rt0), then gemm_split_reduce_kernel with NT_E tiles per workgroup. e0 marks the
// product's start, e1 the reduction's end.
template <int NT, int NB, int EP, int NT_E>
static hipError_t launch_split_t(const GemmParams &p, int row_tiles, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    constexpr int ROWS = kMaxRows, COLS = 16 * NT;
    constexpr bool ROWSCALE = EP != E_RESID && EP != E_LOGITS;
    if (!p.spart || (ROWSCALE && !p.sinv) || row_tiles < 1 || (p.rt0 + row_tiles) * ROWS > p.rr.cap ||
        p.lda % 32 != 0 || p.cols % 16 != 0 || p.Ks < 4 || p.kc != 0)
        return hipErrorInvalidValue;
    GemmParams q = p;
    q.n_wg = (p.cols + COLS - 1) / COLS;
    q.row_tiles = row_tiles;
    const size_t lds = (size_t)split_lds_floats<4, NT, NB>() * sizeof(float);
    const dim3 grid((unsigned)((q.n_wg + 1) / 2 * 8 * row_tiles));
    auto split = gemm_split_kernel<NT, NB, EP>;
    if (e0)
        hipExtLaunchKernelGGL(split, grid, dim3(kGemmWaves * kWave), lds, s, e0, nullptr, 0, q);
    else
        hipLaunchKernelGGL(split, grid, dim3(kGemmWaves * kWave), lds, s, q);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    GemmParams r = p;
    r.n_wg = (p.cols + 16 * NT_E - 1) / (16 * NT_E);
    r.row_tiles = row_tiles;
    const size_t lds_r = (size_t)split_reduce_lds_floats<NT_E, EP>() * sizeof(float);
    const dim3 grid_r((unsigned)r.n_wg, (unsigned)r.row_tiles);
    auto red = gemm_split_reduce_kernel<NT_E, EP>;
    if (e1)
        hipExtLaunchKernelGGL(red, grid_r, dim3(kGemmWaves * kWave), lds_r, s, nullptr, e1, 0, r);
    else
        hipLaunchKernelGGL(red, grid_r, dim3(kGemmWaves * kWave), lds_r, s, r);
    return hipGetLastError();
}

// The residual epilogue of a prompt product: the fp32 partial planes of its NS K ranges summed in
// range order, X += Y, the next RMSNorm operand X (.) gain, the row's RMSNorm factor and, where
// asked for, the per-16-column sums of squares. One workgroup per row (its sum of squares needs no
// second pass): each thread takes the row's 8-column vectors tid, tid + threads, ...; the threads'
// sums are added in a fixed tree (lanes, then waves in order), so the factor depends on the row
// and the model's width only.
template <int NS>
__global__ __launch_bounds__(512) void prompt_reduce_kernel(GemmParams p, size_t zstride) {
    constexpr Prec P = Prec::BF16;
    const int row = blockIdx.x, tid = threadIdx.x;
    request_together(p.rr.tab, p.part, p.Xout, p.gain, p.An, p.ldx, p.cols, p.rr.cap);
    if (row >= p.rr.tab->R) return;
    __shared__ float s_sum[8];
    float ss_row = 0.0f;
    for (int g = tid; g < p.cols / 8; g += blockDim.x) {
        const int c0 = 8 * g;
        const size_t o = (size_t)row * p.ldx + c0;
        f32x4 q[NS][2], xv[2], gv[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int z = 0; z < NS; ++z) q[z][h] = *reinterpret_cast<const f32x4 *>(p.part + z * zstride + o + 4 * h);
            xv[h] = *reinterpret_cast<const f32x4 *>(p.Xout + o + 4 * h);
            gv[h] = *reinterpret_cast<const f32x4 *>(p.gain + c0 + 4 * h);
        }
        alignas(16) float x[8], a[8];
        float ss = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float y = q[0][e >> 2][e & 3];
            if constexpr (NS > 1) y += q[1][e >> 2][e & 3];
            if constexpr (NS == 3) y += q[2][e >> 2][e & 3];
            if constexpr (NS == 4) y += q[2][e >> 2][e & 3] + q[3][e >> 2][e & 3];
            x[e] = xv[e >> 2][e & 3] + y;
            ss += x[e] * x[e];
            a[e] = x[e] * gv[e >> 2][e & 3];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
            *reinterpret_cast<f32x4 *>(p.Xout + o + 4 * h) = *reinterpret_cast<const f32x4 *>(x + 4 * h);
        put_act8(reinterpret_cast<uint16_t *>(p.An), act_plane(p.rr.cap, p.ldx), act_idx<P>(row, c0, p.ldx), a);
        if (p.ssq_out) {  // a 16-column tile is two consecutive threads'
            const float other = __shfl_xor(ss, 1);
            if ((g & 1) == 0) p.ssq_out[(size_t)row * p.T + (g >> 1)] = ss + other;
        }
        ss_row += ss;
    }
    const float inv = row_factor_of_block(ss_row, p.K, p.eps, s_sum);
    if (tid == 0) p.sinv[row] = inv;
}

static hipError_t launch_prompt_reduce(const GemmParams &p, int nsplit, size_t zstride, int rows, hipStream_t s,
                                       hipEvent_t e1) {
    if (!p.sinv || !p.gain || p.cols % 16 != 0) return hipErrorInvalidValue;
    // whole waves, at most 512 threads: one 8-column vector each up to 4096 columns (with 256
    // threads, two vectors each, the 512-row down reduction took 18 us)
    const int threads = std::min(512, (p.cols / 8 + kWave - 1) / kWave * kWave);
    auto kern = nsplit == 1 ? prompt_reduce_kernel<1> : nsplit == 2 ? prompt_reduce_kernel<2>
                : nsplit == 3 ? prompt_reduce_kernel<3> : prompt_reduce_kernel<4>;
    if (e1)
        hipExtLaunchKernelGGL(kern, dim3(rows), dim3(threads), 0, s, nullptr, e1, 0, p, zstride);
    else
        hipLaunchKernelGGL(kern, dim3(rows), dim3(threads), 0, s, p, zstride);
    return hipGetLastError();
}

// The prompt product over `rows` rows; NS > 0 (E_LOGITS): as NS K ranges into the fp32 partial
// planes of p.part, then prompt_reduce_kernel.
template <int NT, int RG, int WM, int EP, int NB, int NS = 0>
static hipError_t launch_prompt_t(const GemmParams &p, int rows, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    constexpr int ROWS = 16 * RG, COLS = 16 * NT;
    constexpr size_t lds = (size_t)prompt_lds_bytes<NT, RG, WM, EP, NB>();
    static_assert(lds <= 160 * 1024, "the LDS of a CU");
    static_assert((NS > 0) == (EP == E_LOGITS) && NS <= kDownSplits, "K ranges");
    if (rows < 1 || rows > p.rr.cap || p.rr.cap % ROWS != 0 || p.lda % 32 != 0 || p.cols % 16 != 0 || p.Ks < 1)
        return hipErrorInvalidValue;
    if (EP == E_LOGITS ? (!p.part || p.ldx < p.cols || p.ldx % 8 != 0) : !p.sinv) return hipErrorInvalidValue;
    if (EP == E_QKV && (p.hd % 16 != 0 || p.d % p.hd != 0)) return hipErrorInvalidValue;
    GemmParams q = p;
    int nsplit = 1;
    if constexpr (NS > 0) {
        q.kc = (p.Ks + NS - 1) / NS;
        nsplit = (p.Ks + q.kc - 1) / q.kc;
        q.Zout = p.part;
        q.ldz = p.ldx;
        q.zstride = (size_t)p.rr.cap * p.ldx;
    }
    q.n_wg = (p.cols + COLS - 1) / COLS;
    q.row_tiles = (rows + ROWS - 1) / ROWS;
    const dim3 grid((unsigned)((q.n_wg + 7) / 8 * 8 * q.row_tiles), (unsigned)nsplit);  // column groups padded to 8 XCDs
    auto kern = gemm_prompt_kernel<NT, RG, WM, EP, NB>;
    hipEvent_t end = NS > 0 ? nullptr : e1;
    if (e0 || end)
        hipExtLaunchKernelGGL(kern, grid, dim3(kGemmWaves * kWave), lds, s, e0, end, 0, q);
    else
        hipLaunchKernelGGL(kern, grid, dim3(kGemmWaves * kWave), lds, s, q);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess || NS == 0) return err;
    return launch_prompt_reduce(p, nsplit, q.zstride, rows, s, e1);
}

// Tile rule of the prompt products: the tile whose launch should take the least time, a + b rounds.
// A round is one workgroup per CU (32 on an XCD, which holds the column groups cg with cg % 8 its
// number: 20 groups are three on four of the XCDs and two on the others); b is the time of a
// round and a what the first one adds (ramp; the smaller tiles, two of which share a CU, hide part
// of the later ones' latency). A second, partly filled round costs as much as a full one, and a
// larger tile than needed leaves CUs idle while its workgroups take longer. The constants are us at
// 128 k-steps, fitted to forced-tile sweeps over d 2048, 3072, 4096 and 5120 and 64 to 2048 rows;
// time is nearly proportional to the k-steps for every tile, so the choice does not depend on them.
// A row's values do not depend on the tile. Of the sweep's 208 launches the rule takes the fastest tile,
// or one within 2%, but for five (at most 6% off). Against the former rule (the smallest tile whose
// workgroups are one round, else the largest), us a launch: d 5120, 512 rows gate/up 313 -> 273, down
// 156 -> 141; 192 rows gate/up 148 -> 121; 320 rows down 137 -> 97; d 4096, 640 rows gate/up 253 ->
// 220; d 3072, 640 rows down 94 -> 66. At the 7B widths up to 512 rows the two choose alike.
struct PromptTile {
    int nt, rg;  // 16 nt columns x 16 rg rows
    float a, b;
};
template <size_t N>
static int prompt_tile(const PromptTile (&tiles)[N], const GemmParams &p, int rows, int splits) {
    int best = 0;
    float least = 0.0f;
    for (int i = 0; i < (int)N; ++i) {
        const PromptTile &t = tiles[i];
        const int groups = (p.cols + 16 * t.nt - 1) / (16 * t.nt), row_tiles = (rows + 16 * t.rg - 1) / (16 * t.rg);
        const int per_xcd = (groups + 7) / 8 * row_tiles * splits;
        const float cost = t.a + t.b * (float)((per_xcd + kCUs / 8 - 1) / (kCUs / 8));
        if (i == 0 || cost < least) least = cost, best = i;
    }
    return best;
}

constexpr int kPromptSplitsO = 2, kPromptSplitsDown = 4;

template <int NS>
static hipError_t launch_prompt_resid(const GemmParams &p, int rows, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    static const PromptTile tiles[] = {{4, 4, 8.0f, 16.7f}, {8, 4, 8.5f, 22.0f}, {8, 8, 2.0f, 41.5f}, {16, 8, 2.0f, 66.0f}};
    switch (prompt_tile(tiles, p, rows, NS)) {
    case 0: return launch_prompt_t<4, 4, 2, E_LOGITS, 5, NS>(p, rows, s, e0, e1);
    case 1: return launch_prompt_t<8, 4, 2, E_LOGITS, 5, NS>(p, rows, s, e0, e1);
    case 2: return launch_prompt_t<8, 8, 2, E_LOGITS, 5, NS>(p, rows, s, e0, e1);
    default: return launch_prompt_t<16, 8, 2, E_LOGITS, 4, NS>(p, rows, s, e0, e1);
    }
}

static hipError_t launch_prompt_qkv(const GemmParams &p, int rows, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    static const PromptTile tiles[] = {{4, 4, 10.0f, 23.5f}, {6, 4, 13.0f, 27.0f}, {12, 4, 3.0f, 48.0f}, {12, 8, 0.0f, 78.0f}};
    switch (prompt_tile(tiles, p, rows, 1)) {
    case 0: return launch_prompt_t<4, 4, 2, E_QKV, 5>(p, rows, s, e0, e1);
    case 1: return launch_prompt_t<6, 4, 4, E_QKV, 5>(p, rows, s, e0, e1);
    case 2: return launch_prompt_t<12, 4, 2, E_QKV, 5>(p, rows, s, e0, e1);
    default: return launch_prompt_t<12, 8, 2, E_QKV, 5>(p, rows, s, e0, e1);
    }
}

static hipError_t launch_prompt_gate_up(const GemmParams &p, int rows, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    static const PromptTile tiles[] = {{4, 4, 10.0f, 24.5f}, {8, 4, 14.0f, 29.5f}, {12, 4, 8.0f, 45.0f}, {12, 8, 0.0f, 78.0f},
                                       {24, 8, 0.0f, 126.0f}};
    switch (prompt_tile(tiles, p, rows, 1)) {
    case 0: return launch_prompt_t<4, 4, 4, E_SWIGLU, 5>(p, rows, s, e0, e1);
    case 1: return launch_prompt_t<8, 4, 2, E_SWIGLU, 5>(p, rows, s, e0, e1);
    case 2: return launch_prompt_t<12, 4, 4, E_SWIGLU, 5>(p, rows, s, e0, e1);
    case 3: return launch_prompt_t<12, 8, 4, E_SWIGLU, 5>(p, rows, s, e0, e1);
    default: return launch_prompt_t<24, 8, 2, E_SWIGLU, 4>(p, rows, s, e0, e1);
    }
}

// O and down split K into 2 and 4 ranges (fixed: they are part of a row's reduction order), which
// gives their 4096 columns as many workgroups at 512 rows as the other products have.
hipError_t launch_gemm_prompt(GemmKind kind, int rows, const GemmParams &p, hipStream_t s, hipEvent_t e0,
                              hipEvent_t e1) {
    switch (kind) {
    case GEMM_QKV: return launch_prompt_qkv(p, rows, s, e0, e1);
    case GEMM_GATE_UP: return launch_prompt_gate_up(p, rows, s, e0, e1);
    case GEMM_O: return launch_prompt_resid<kPromptSplitsO>(p, rows, s, e0, e1);        // X += O W_o^T
    case GEMM_DOWN: return launch_prompt_resid<kPromptSplitsDown>(p, rows, s, e0, e1);  // X += H W_d^T
    default: return hipErrorInvalidValue;
    }
}

// Plain fp32 product of a few rows (the loss head's logits and dH, bf16): the prompt kernel's
// tiles over `rows` <= 128 rows, with p.kc > 0 as K ranges into planes of p.Zout.
template <int NT, int RG, int WM, int NB>
static hipError_t launch_rows_product_t(const GemmParams &p, int rows, int splits, hipStream_t s, hipEvent_t e0,
                                        hipEvent_t e1) {
    constexpr int ROWS = 16 * RG, COLS = 16 * NT;
    constexpr size_t lds = (size_t)prompt_lds_bytes<NT, RG, WM, E_LOGITS, NB, true>();
    static_assert(lds <= 160 * 1024, "the LDS of a CU");
    if (rows > ROWS || p.rr.cap < ROWS) return hipErrorInvalidValue;
    GemmParams q = p;
    q.n_wg = (p.cols + COLS - 1) / COLS;
    q.row_tiles = 1;
    const dim3 grid((unsigned)((q.n_wg + 7) / 8 * 8), (unsigned)splits);
    auto kern = gemm_prompt_kernel<NT, RG, WM, E_LOGITS, NB, true>;
    if (e0 || e1)
        hipExtLaunchKernelGGL(kern, grid, dim3(kGemmWaves * kWave), lds, s, e0, e1, 0, q);
    else
        hipLaunchKernelGGL(kern, grid, dim3(kGemmWaves * kWave), lds, s, q);
    return hipGetLastError();
}

// Up to 64, 96 and 128 rows take tiles of as many rows x 128 columns: the 7B head's 32000 columns are
// then 250 workgroups, one round of the CUs, and the head is streamed once for all rows (two launches
// of gemm_kernel, one per 64-row tile, took 104 us for 80 rows of it). The class accumulators cost
// 3-4% of a whole call in 128-row tiles, whose ring is then four buffers (7B head, 64 pairs without
// dW: 176 -> 183 us), and up to 2% in 64-row ones. The 96-row tile, which holds five buffers, gives
// that back (16 pairs and 48 AR rows: 170 us with one chain, 177 in a 128-row tile, 169 in a 96-row one).
//
// Few rows take gemm_kernel, which skips the row groups that hold none and has two workgroups per CU
// to hide a short row's latency; a 64-row tile reads and multiplies its padding (one pair, whole
// call, tile against gemm_kernel: 7B head 133 -> 117 us, vocabulary 128256 420 -> 359, 8192 x 2048
// 58 -> 51). The logits change over above 16 rows (20 rows: 127 us in tiles, 132 with gemm_kernel),
// dH's K ranges, whose workgroups are shorter, above 32 (20 rows: 136 with gemm_kernel, 138 in tiles;
// above 32 gemm_kernel is 5-9% slower).
constexpr int kFewRows = 16, kFewRowsSplit = 32;

hipError_t launch_rows_product(int rows, const GemmParams &p, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    if (rows < 1 || rows > 128 || rows > p.rr.cap || p.lda % 32 != 0 || p.cols % 16 != 0 || p.Ks < 1 || p.kc < 0 ||
        !p.Zout || p.ldz < p.cols || p.ldz % 4 != 0 || p.zstride % 4 != 0)
        return hipErrorInvalidValue;
    if (rows <= (p.kc > 0 ? kFewRowsSplit : kFewRows))
        return launch_gemm(GEMM_LOGITS, true, rows <= 16 ? 1 : 2, 1, p, s, e0, e1);
    const int splits = p.kc > 0 ? (p.Ks + p.kc - 1) / p.kc : 1;
    if (rows <= 64) return launch_rows_product_t<8, 4, 2, 5>(p, rows, splits, s, e0, e1);
    if (rows <= 96) return launch_rows_product_t<8, 6, 2, 5>(p, rows, splits, s, e0, e1);
    return launch_rows_product_t<8, 8, 2, 4>(p, rows, splits, s, e0, e1);
}

// Grid: column workgroups (ceil(p.cols / (16 * NT))) x row tiles of 16 * RG rows (from row tile
// p.rt0) x K splits (E_LOGITS with p.kc > 0).
template <Prec P, int NT, int RG, int EP, int D = kGemmDepth, int W = kGemmWaves>
static hipError_t launch_gemm_t(const GemmParams &p, int row_tiles, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    constexpr int ROWS = 16 * RG, COLS = 16 * NT;
    static_assert(W * NT * 256 >= ROWS * COLS, "E_RESID reuses the reduction buffer");
    const size_t lds = (size_t)tile_lds_floats<NT, RG, W>() * sizeof(float);
    auto kern = row_tiles > 1 ? gemm_kernel<P, NT, RG, EP, D, W, true> : gemm_kernel<P, NT, RG, EP, D, W, false>;
    GemmParams q = p;
    q.row_tiles = row_tiles;
    q.n_wg = (p.cols + COLS - 1) / COLS;  // the last workgroup may be ragged
    const int splits = EP == E_LOGITS && p.kc > 0 ? (p.Ks + p.kc - 1) / p.kc : 1;
    if (EP != E_LOGITS && p.kc != 0) return hipErrorInvalidValue;
    const dim3 grid(q.n_wg, row_tiles, splits);
    if (e0 || e1) {
        hipExtLaunchKernelGGL(kern, grid, dim3(W * kWave), lds, s, e0, e1, 0, q);
    } else {
        hipLaunchKernelGGL(kern, grid, dim3(W * kWave), lds, s, q);
    }
    return hipGetLastError();
}

// The down product's epilogue: the K-split partial products of kDownSplits workgroups per
// column group summed in a fixed tree, (p0 + p1) + (p2 + p3) (splits past the last are absent
// terms), then X += Y, the next RMSNorm operand X (.) gain (one operand vector per thread) and
// the per-16-column sums of squares: each thread sums its VEC columns in order, the threads of
// a 16-column tile then add their sums in order. Rows past the iteration's rows (device row
// table) exit.
constexpr int kReduceThreads = 64;  // one wave per workgroup: the reduction is latency-bound

template <Prec P>
__global__ __launch_bounds__(kReduceThreads) void down_reduce_kernel(GemmParams p, int nsplit, size_t zstride, int rows_launch) {
    using PT = PrecT<P>;
    using T = typename PT::T;
    constexpr int VEC = PT::VEC, G = 16 / VEC;  // columns per thread, threads per 16-column tile
    const int groups = p.cols / VEC;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int row = (int)(i / groups), g = (int)(i % groups);  // G consecutive threads share a tile
    const bool live = row < rows_launch && row < p.rr.tab->R;
    float ss = 0.0f;
    if (live) {
        const int c0 = g * VEC;
        const size_t o = (size_t)row * p.ldx + c0;
        float y[VEC], x[VEC];
#pragma unroll
        for (int h = 0; h < VEC / 4; ++h) {
            f32x4 q[kDownSplits];
#pragma unroll
            for (int z = 0; z < kDownSplits; ++z)
                q[z] = z < nsplit ? *reinterpret_cast<const f32x4 *>(p.part + z * zstride + o + 4 * h)
                                  : f32x4{0.f, 0.f, 0.f, 0.f};
            const f32x4 xv = *reinterpret_cast<const f32x4 *>(p.Xout + o + 4 * h);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                y[4 * h + e] = (q[0][e] + q[1][e]) + (q[2][e] + q[3][e]);
                x[4 * h + e] = xv[e] + y[4 * h + e];
            }
        }
        alignas(16) T hi[VEC], lo[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            ss += x[e] * x[e];
            const float a = x[e] * p.gain[c0 + e];
            if constexpr (P == Prec::BF16) {
                hi[e] = f2bf(a);
                lo[e] = f2bf(a - bf2f(hi[e]));
            } else {
                hi[e] = a;
            }
        }
#pragma unroll
        for (int h = 0; h < VEC / 4; ++h)
            *reinterpret_cast<f32x4 *>(p.Xout + o + 4 * h) = f32x4{x[4 * h], x[4 * h + 1], x[4 * h + 2], x[4 * h + 3]};
        T *an = reinterpret_cast<T *>(p.An);
        const size_t ai = act_idx<P>(row, c0, p.ldx);  // VEC consecutive columns: one operand vector
        *reinterpret_cast<u32x4 *>(an + ai) = *reinterpret_cast<const u32x4 *>(hi);
        if constexpr (P == Prec::BF16)
            *reinterpret_cast<u32x4 *>(an + act_plane(p.rr.cap, p.ldx) + ai) = *reinterpret_cast<const u32x4 *>(lo);
    }
    // the tile's G partial sums in order (G consecutive lanes; every lane takes part)
    float tot = 0.0f;
    const int base = (threadIdx.x & 63) & ~(G - 1);
#pragma unroll
    for (int k = 0; k < G; ++k) tot += __shfl(ss, base + k);
    if (live && g % G == 0) p.ssq_out[(size_t)row * p.T + g / G] = tot;
}

// The down product: K split over kDownSplits ranges (fp32 partials in p.part, 64-column
// workgroups, D k-steps in flight), then down_reduce_kernel. e0 marks the product's start, e1
// the reduction's end.
// ROWK: the split products through the row-tiled kernel (bf16, several row tiles; the same values
// as gemm_kernel's).
template <Prec P, int RG, int D, bool ROWK = false>
static hipError_t launch_down(const GemmParams &p, int row_tiles, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    static_assert(kDownSplits == 4, "down_reduce_kernel sums four partials");
    if (!p.part || p.rt0 != 0 || p.cols % 16 != 0 || p.ldx < p.cols) return hipErrorInvalidValue;
    GemmParams q = p;
    q.kc = (p.Ks + kDownSplits - 1) / kDownSplits;
    q.Zout = p.part;
    q.ldz = p.ldx;
    q.V = p.cols;
    q.zstride = (size_t)p.rr.cap * p.ldx;
    hipError_t err;
    if constexpr (ROWK)
        err = launch_rows_t<kRowsNtDown, E_LOGITS, kRowsNbDown, kLmTiles, D>(q, row_tiles, s, e0, nullptr);
    else
        err = launch_gemm_t<P, kLmTiles, RG, E_LOGITS, D>(q, row_tiles, s, e0, nullptr);
    if (err != hipSuccess) return err;
    const int nsplit = (p.Ks + q.kc - 1) / q.kc;
    const int rows_launch = row_tiles * 16 * RG;
    const size_t n = (size_t)rows_launch * (p.cols / PrecT<P>::VEC);
    const dim3 grid((unsigned)((n + kReduceThreads - 1) / kReduceThreads));
    if (e1)
        hipExtLaunchKernelGGL(down_reduce_kernel<P>, grid, dim3(kReduceThreads), 0, s, nullptr, e1, 0, p, nsplit, q.zstride,
                              rows_launch);
    else
        hipLaunchKernelGGL(down_reduce_kernel<P>, grid, dim3(kReduceThreads), 0, s, p, nsplit, q.zstride, rows_launch);
    return hipGetLastError();
}

// Small models: a launch whose K is at most kShortKs k-steps (eight per wave) is a latency chain, not
// a stream. It takes the smallest column tile whose workgroups fit the CUs in one round (more CUs
// pull, and a workgroup's tree and epilogue are shorter) with up to four k-steps of a wave in flight,
// which at K = 768 is all of them. The k-steps of a wave and the tree are the same for every tile
// and depth, so the values are those of the larger tiles. Measured at d 768, FFN 2048 (one row,
// us a launch): QKV 6.0 -> 5.0 (tiles of 48 -> 16 columns: 48 -> 144 workgroups), gate/up 7.0 ->
// 5.2 (96 -> 32: 43 -> 128), down with its reduction 6.2 and a launch gap -> 5.2. Above 64 k-steps
// the larger tiles and the K ranges stay: the launch is a stream there (d 4096: QKV 256 workgroups
// with the larger tile already, down 21.5 us in one launch against 19.1 with its reduction). Between
// 65 and 128 k-steps it depends on the rows, which the order of a sum must not: an iteration of a
// model with FFN 2080 to 4096 would gain 4-10% at 1 and 16 rows with the line at 128 and lose 3-7% at
// 64 (d 1024, FFN 4096: 352 -> 334 us at one row, 504 -> 545 at 64).
constexpr int kShortKs = 64, kShortDepth = 4;

// The down product of such a K is one launch, without K ranges and their reduction. The rule reads
// the model's shape only: every row count takes the same order. Over several row tiles it takes
// 16-column tiles while they are one round of the CUs, else 32-column ones: the 64-column tiles that the
// K ranges had would be few workgroups walking all of K. Batched decoding of a fp32 model (4 layers, d
// 256, FFN 688), 32 sequences x 16 rows, ms: 13.5 with K ranges, 15.1 in 64-column tiles, 12.9 in
// 16-column ones; 12 layers of d 768: 35.5, 33.7, 32.4; d 1024, 64 x 16 rows (1024 workgroups of 16
// columns): 33.4 in 64-column tiles, 33.8 in 16-, 32.7 in 32-column ones.
static bool short_k(const GemmParams &p) { return p.Ks <= kShortKs; }
static bool one_round(const GemmParams &p, int nt, int row_tiles = 1) {
    return ((p.cols >> 4) + nt - 1) / nt * row_tiles <= kCUs;
}

template <Prec P, int RG>
static hipError_t launch_gemm_rg(GemmKind kind, const GemmParams &p, int row_tiles, hipStream_t s, hipEvent_t e0,
                                 hipEvent_t e1) {
    if (row_tiles > 1 && P == Prec::BF16 && !p.tile_kernel && p.spart && p.Ks >= 4) {
        // More than 64 rows, bf16 (K of at least four k-steps): QKV, gate/up and the LM head
        // through the class-pair K split (the same values)
        if (kind == GEMM_QKV)
            return launch_split_t<kSplitNtQkv, kSplitNbQkv, E_QKV, 4>(p, row_tiles, s, e0, e1);
        if (kind == GEMM_GATE_UP)
            return launch_split_t<kSplitNtGateUp, kSplitNbGateUp, E_SWIGLU, 4>(p, row_tiles, s, e0, e1);
        // the reduction's column groups are the LM head's argmax workgroups (kLmTiles tiles each)
        if (kind == GEMM_LM)
            return launch_split_t<kSplitNtLm, kSplitNbLm, E_ARGMAX, kLmTiles>(p, row_tiles, s, e0, e1);
    }
    if (row_tiles > 1 && P == Prec::BF16 && !p.tile_kernel) {
        // More than 64 rows, bf16: gate/up and the down product take the row-tiled kernel (the
        // same values); at 7B, 96 / 160 / 256 / 512 rows: gate/up 59 / 112 / 115 / 221 us against
        // 77 / 110 / 144 / 278, down (with its reduction) 36 / 62 / 62 / 116 against 46 / 62 / 80 / 143
        if (kind == GEMM_GATE_UP) return launch_rows_t<kRowsNtGateUp, E_SWIGLU, kRowsNbGateUp, 6, 2>(p, row_tiles, s, e0, e1);
        if (kind == GEMM_DOWN && !short_k(p)) return launch_down<P, RG, 3, true>(p, row_tiles, s, e0, e1);
    }
    if (row_tiles > 1) {
        // More than 64 rows (measured at 160 and 512 rows, 7B): QKV and gate/up take 96-column
        // workgroups (two k-steps in flight), O and down 64-column workgroups (three k-steps in
        // flight). Row tiles past the iteration's rows exit at once, so a batched iteration
        // launched for its largest row count costs what its live rows cost.
        switch (kind) {
        case GEMM_QKV:
            return launch_gemm_t<P, 6, RG, E_QKV, 2>(p, row_tiles, s, e0, e1);
        case GEMM_O:
            return launch_gemm_t<P, 4, RG, E_RESID, 3>(p, row_tiles, s, e0, e1);
        case GEMM_DOWN:
            if (short_k(p)) {
                if (one_round(p, 1, row_tiles)) return launch_gemm_t<P, 1, RG, E_RESID, 3>(p, row_tiles, s, e0, e1);
                return launch_gemm_t<P, 2, RG, E_RESID, 3>(p, row_tiles, s, e0, e1);
            }
            return launch_down<P, RG, 3>(p, row_tiles, s, e0, e1);
        case GEMM_GATE_UP:
            return launch_gemm_t<P, 6, RG, E_SWIGLU, 2>(p, row_tiles, s, e0, e1);
        case GEMM_LM:
            return launch_gemm_t<P, kLmTiles, RG, E_ARGMAX, 3>(p, row_tiles, s, e0, e1);
        case GEMM_LOGITS:
            return launch_gemm_t<P, kLmTiles, RG, E_LOGITS, 3>(p, row_tiles, s, e0, e1);
        }
        return hipErrorInvalidValue;
    }
    switch (kind) {
    case GEMM_QKV:
        if (short_k(p) && one_round(p, 1)) return launch_gemm_t<P, 1, RG, E_QKV, kShortDepth>(p, row_tiles, s, e0, e1);
        return launch_gemm_t<P, kNtQkv, RG, E_QKV>(p, row_tiles, s, e0, e1);
    case GEMM_O:
        if (short_k(p)) return launch_gemm_t<P, kNtResid, RG, E_RESID, kShortDepth>(p, row_tiles, s, e0, e1);
        return launch_gemm_t<P, kNtResid, RG, E_RESID>(p, row_tiles, s, e0, e1);
    case GEMM_DOWN:
        if (short_k(p)) return launch_gemm_t<P, kNtResid, RG, E_RESID, kShortDepth>(p, row_tiles, s, e0, e1);
        return launch_down<P, RG, kGemmDepth>(p, row_tiles, s, e0, e1);
    case GEMM_GATE_UP:
        if (short_k(p) && one_round(p, 2)) return launch_gemm_t<P, 2, RG, E_SWIGLU, kShortDepth>(p, row_tiles, s, e0, e1);
        return launch_gemm_t<P, kNtGateUp, RG, E_SWIGLU>(p, row_tiles, s, e0, e1);
    case GEMM_LM:
        return launch_gemm_t<P, kLmTiles, RG, E_ARGMAX>(p, row_tiles, s, e0, e1);
    case GEMM_LOGITS:
        return launch_gemm_t<P, kLmTiles, RG, E_LOGITS>(p, row_tiles, s, e0, e1);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gemm(GemmKind kind, bool bf16, int rg, int row_tiles, const GemmParams &p, hipStream_t s,
                       hipEvent_t e0, hipEvent_t e1) {
    if (row_tiles < 1 || (row_tiles > 1 && rg != 4)) return hipErrorInvalidValue;
    if (bf16) {
        if (rg == 1) return launch_gemm_rg<Prec::BF16, 1>(kind, p, row_tiles, s, e0, e1);
        if (rg == 2) return launch_gemm_rg<Prec::BF16, 2>(kind, p, row_tiles, s, e0, e1);
        return launch_gemm_rg<Prec::BF16, 4>(kind, p, row_tiles, s, e0, e1);
    }
    if (rg == 1) return launch_gemm_rg<Prec::F32, 1>(kind, p, row_tiles, s, e0, e1);
    if (rg == 2) return launch_gemm_rg<Prec::F32, 2>(kind, p, row_tiles, s, e0, e1);
    return launch_gemm_rg<Prec::F32, 4>(kind, p, row_tiles, s, e0, e1);
}

}  // namespace cllm
