// CLLM training loss head on gfx950: the global-consistency and AR losses of Section 3.2.2
// (eqs. global_loss, ar_loss) at the LM head, forward then backward.
//
// Inputs are LM-head input rows H (fp32): P teacher rows (conditioned on the fixed point y*,
// stop-gradient), P student rows (on the trajectory state y at the same positions) and A rows of
// the target model's generation with their target ids. The logits Z = H W^T come from
// launch_rows_product (bf16) or gemm_kernel (fp32), E_LOGITS epilogue. Per pair the loss is the forward KL D(p || q) between
// p = softmax(teacher logits) and q = softmax(student logits); per AR row -log softmax at the
// target; L = sum KL + omega sum NLL. Backward: D = dL/dZ for the student and AR rows
// (q - p; omega (softmax - onehot)), dH = D W (the same products, over a transposed copy
// of the packed LM head, K split across workgroups) and dW = D^T H (teacher rows get no
// gradient). In bf16 the fp32 operands D and H enter the MFMAs as hi + lo bf16 planes, as the
// activations of the forward do. Every sum has a fixed order (per-thread strided runs, fixed
// shuffle and wave trees, vocabulary chunks and K splits in index order), so results do not
// depend on timing.
#include <hip/hip_ext.h>

#include "device.h"
#include "launch.h"

namespace cllm {

namespace {

constexpr int kLossThreads = 256;
constexpr int kStat = 5;  // statistics per (row, chunk): pair (ma, za, cross, ms, zs); AR (mc, zc)

// Sum / max over a 256-thread workgroup in a fixed order (xor tree inside each wave, then the
// four waves in order); every thread gets the result.
template <bool MAX>
__device__ float block_reduce(float v, float *s_buf) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const float o = __shfl_xor(v, off);
        v = MAX ? fmaxf(v, o) : v + o;
    }
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s_buf[w] = v;
    __syncthreads();
    return MAX ? fmaxf(fmaxf(s_buf[0], s_buf[1]), fmaxf(s_buf[2], s_buf[3]))
               : (s_buf[0] + s_buf[1]) + (s_buf[2] + s_buf[3]);
}

// Eight fp32 values as the hi and lo bf16 vectors of an MFMA operand (lo = bf16(x - hi)).
__device__ __forceinline__ void split8(const float (&x)[8], u32x4 &hi, u32x4 &lo) {
    uint32_t h[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint16_t h0 = f2bf(x[2 * i]), h1 = f2bf(x[2 * i + 1]);
        const uint16_t l0 = f2bf(x[2 * i] - bf2f(h0)), l1 = f2bf(x[2 * i + 1] - bf2f(h1));
        h[i] = (uint32_t)h0 | ((uint32_t)h1 << 16);
        l[i] = (uint32_t)l0 | ((uint32_t)l1 << 16);
    }
    hi = u32x4{h[0], h[1], h[2], h[3]};
    lo = u32x4{l[0], l[1], l[2], l[3]};
}

// Operand order of an [n][r] matrix whose contraction index is r (rpad rows, zero past the
// data): for 16-row group n/16 and k-step r/32, lane 16 * ((r % 32) / 8) + n % 16, element r % 8.
__device__ __forceinline__ size_t tr_idx(int n, int r, int ks) {
    return ((size_t)((n >> 4) * ks + (r >> 5)) * kWave + 16 * ((r & 31) >> 3) + (n & 15)) * 8 + (r & 7);
}

}  // namespace

// Row statistics, phase 1: workgroup (chunk c of kLossChunk vocabulary entries, row item b); item
// b < P is pair b (teacher row b, student row P + b), item P + i is AR row i.
__global__ __launch_bounds__(kLossThreads) void loss_stats_kernel(LossParams p, float *stats, int nch) {
    __shared__ float s_buf[4];
    const int c = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int v0 = c * kLossChunk, v1 = min(v0 + kLossChunk, p.V);
    float *st = stats + ((size_t)b * nch + c) * kStat;
    if (b < p.P) {
        const float *a = p.Z + (size_t)b * p.ldz, *s = p.Z + (size_t)(p.P + b) * p.ldz;
        float ma = -INFINITY, ms = -INFINITY;
        for (int v = v0 + tid; v < v1; v += kLossThreads) {
            ma = fmaxf(ma, a[v]);
            ms = fmaxf(ms, s[v]);
        }
        ma = block_reduce<true>(ma, s_buf);
        ms = block_reduce<true>(ms, s_buf);
        float za = 0.f, zs = 0.f, cross = 0.f;
        for (int v = v0 + tid; v < v1; v += kLossThreads) {
            const float ea = expf(a[v] - ma);
            za += ea;
            zs += expf(s[v] - ms);
            cross += ea * (a[v] - s[v]);
        }
        za = block_reduce<false>(za, s_buf);
        zs = block_reduce<false>(zs, s_buf);
        cross = block_reduce<false>(cross, s_buf);
        if (tid == 0) {
            st[0] = ma;
            st[1] = za;
            st[2] = cross;
            st[3] = ms;
            st[4] = zs;
        }
    } else {
        const float *z = p.Z + (size_t)(2 * p.P + b - p.P) * p.ldz;
        float mc = -INFINITY;
        for (int v = v0 + tid; v < v1; v += kLossThreads) mc = fmaxf(mc, z[v]);
        mc = block_reduce<true>(mc, s_buf);
        float zc = 0.f;
        for (int v = v0 + tid; v < v1; v += kLossThreads) zc += expf(z[v] - mc);
        zc = block_reduce<false>(zc, s_buf);
        if (tid == 0) {
            st[0] = mc;
            st[1] = zc;
        }
    }
}

// Row statistics, phase 2 (fp32): the chunks' statistics combined in chunk order (every thread the
// same), then the row's loss (chunk 0) and its logit gradients over the chunk (0 past V).
__global__ __launch_bounds__(kLossThreads) void loss_grad_kernel(LossParams p, const float *stats, int nch) {
    const int c = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int V = p.V, v0 = c * kLossChunk, v1 = min(v0 + kLossChunk, p.ldz);
    const float *st = stats + (size_t)b * nch * kStat;
    if (b < p.P) {
        float ma = -INFINITY, ms = -INFINITY;
        for (int q = 0; q < nch; ++q) {
            ma = fmaxf(ma, st[q * kStat + 0]);
            ms = fmaxf(ms, st[q * kStat + 3]);
        }
        float za = 0.f, zs = 0.f, cross = 0.f;
        for (int q = 0; q < nch; ++q) {
            const float fa = expf(st[q * kStat + 0] - ma);
            za += st[q * kStat + 1] * fa;
            cross += st[q * kStat + 2] * fa;
            zs += st[q * kStat + 4] * expf(st[q * kStat + 3] - ms);
        }
        // KL(p || q) = sum_v p_v (a_v - s_v) - logsumexp(a) + logsumexp(s)
        if (c == 0 && tid == 0) p.kl[b] = cross / za - (ma + logf(za)) + (ms + logf(zs));
        const float *a = p.Z + (size_t)b * p.ldz, *s = p.Z + (size_t)(p.P + b) * p.ldz;
        float *d = p.D + (size_t)b * p.ldz;
        const float ia = 1.0f / za, is = 1.0f / zs;
        for (int v = v0 + tid; v < v1; v += kLossThreads)
            d[v] = v < V ? expf(s[v] - ms) * is - expf(a[v] - ma) * ia : 0.0f;
    } else {
        const int i = b - p.P;
        const float *z = p.Z + (size_t)(2 * p.P + i) * p.ldz;
        const int t = p.targets[i];
        float *d = p.D + (size_t)(p.P + i) * p.ldz;
        if (t < 0 || t >= V) {  // a target outside the vocabulary: NaN loss and gradient row
            if (c == 0 && tid == 0) p.nll[i] = NAN;
            for (int v = v0 + tid; v < v1; v += kLossThreads) d[v] = v < V ? NAN : 0.0f;
            return;
        }
        float mc = -INFINITY;
        for (int q = 0; q < nch; ++q) mc = fmaxf(mc, st[q * kStat + 0]);
        float zc = 0.f;
        for (int q = 0; q < nch; ++q) zc += st[q * kStat + 1] * expf(st[q * kStat + 0] - mc);
        if (c == 0 && tid == 0) p.nll[i] = mc + logf(zc) - z[t];
        const float ic = 1.0f / zc;
        for (int v = v0 + tid; v < v1; v += kLossThreads)
            d[v] = v < V ? p.omega * (expf(z[v] - mc) * ic - (v == t ? 1.0f : 0.0f)) : 0.0f;
    }
}

// GEMM rows: teacher rows 0..np-1, student rows np..2np-1, AR rows 2np..2np+na-1.
template <Prec P>
__global__ void pack_rows_kernel(const float *T0, const float *S0, int np, const float *R0, int na, int d, int cap,
                                 void *A) {
    using T = typename PrecT<P>::T;
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)(2 * np + na) * d) return;
    const int r = (int)(i / d), k = (int)(i % d);
    const float x = r < np ? T0[(size_t)r * d + k] : r < 2 * np ? S0[(size_t)(r - np) * d + k]
                                                                 : R0[(size_t)(r - 2 * np) * d + k];
    put_act<P>(reinterpret_cast<T *>(A), act_plane(cap, d), act_idx<P>(r, k, d), x);
}

// The same for bf16, eight columns per thread, in one launch with the rows of dW = D^T H (student
// rows S0, then AR rows R0; zero to rpad) as the operand with contraction over the rows: HT, two
// planes of d x rpad, thread (column, 8 rows). The first n_rows workgroups pack the GEMM rows.
__global__ __launch_bounds__(256) void pack_inputs_kernel(const float *T0, const float *S0, int np, const float *R0,
                                                          int na, int d, int cap, uint16_t *A, int n_rows, int rpad,
                                                          uint16_t *HT) {
    if ((int)blockIdx.x < n_rows) {
        const int i = blockIdx.x * 256 + threadIdx.x, r = i / (d / 8), k = i % (d / 8) * 8;
        if (r >= 2 * np + na) return;
        const float *src = r < np ? T0 + (size_t)r * d : r < 2 * np ? S0 + (size_t)(r - np) * d : R0 + (size_t)(r - 2 * np) * d;
        float x[8];  // the caller's arrays: 4-byte alignment is all that is known
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = src[k + e];
        put_act8(A, act_plane(cap, d), act_idx<Prec::BF16>(r, k, d), x);
        return;
    }
    const int t = (blockIdx.x - n_rows) * 256 + threadIdx.x, k = t % d, r0 = t / d * 8, rows = np + na;
    if (r0 >= rpad) return;
    float x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = r0 + i;
        x[i] = r >= rows ? 0.f : r < np ? S0[(size_t)r * d + k] : R0[(size_t)(r - np) * d + k];
    }
    u32x4 h, l;
    split8(x, h, l);
    const size_t o = tr_idx(k, r0, rpad / 32);
    *reinterpret_cast<u32x4 *>(HT + o) = h;
    *reinterpret_cast<u32x4 *>(HT + (size_t)d * rpad + o) = l;
}

// The statistics of n chunks folded in chunk order (PAIR: student logits and the cross term too).
template <bool PAIR>
__device__ __forceinline__ void fold_max(const float *st, int n, float &ma, float &ms) {
    for (int k = 0; k < n; ++k) {
        ma = fmaxf(ma, st[k * kStat + 0]);
        if constexpr (PAIR) ms = fmaxf(ms, st[k * kStat + 3]);
    }
}
template <bool PAIR>
__device__ __forceinline__ void fold_sum(const float *st, int n, float ma, float ms, float &za, float &zs, float &cross) {
    for (int k = 0; k < n; ++k) {
        const float fa = expf(st[k * kStat + 0] - ma);
        za += st[k * kStat + 1] * fa;
        if constexpr (PAIR) {
            cross += st[k * kStat + 2] * fa;
            zs += st[k * kStat + 4] * expf(st[k * kStat + 3] - ms);
        }
    }
}

// Row b's loss from its folded statistics.
__device__ __forceinline__ void write_loss(const LossParams &p, int b, float ma, float ms, float za, float zs, float cross) {
    if (b < p.P) {
        // KL(p || q) = sum_v p_v (a_v - s_v) - logsumexp(a) + logsumexp(s)
        p.kl[b] = cross / za - (ma + logf(za)) + (ms + logf(zs));
    } else {
        const int i = b - p.P, t = p.targets[i];
        // a target outside the vocabulary: NaN
        p.nll[i] = t < 0 || t >= p.V ? NAN : ma + logf(za) - p.Z[(size_t)(2 * p.P + i) * p.ldz + t];
    }
}

// The chunks of each row folded into the first one's place, in chunk order, and the row's loss: one
// wave per row, 64 chunks at a time through LDS.
__global__ __launch_bounds__(kWave) void loss_fold_kernel(LossParams p, float *stats, int nch) {
    __shared__ float s_st[kWave * kStat];
    const int b = blockIdx.x, lane = threadIdx.x;
    const bool pair = b < p.P;
    float *st = stats + (size_t)b * nch * kStat;
    float ma = -INFINITY, ms = -INFINITY, za = 0.f, zs = 0.f, cross = 0.f;
    for (int pass = 0; pass < 2; ++pass)
        for (int q0 = 0; q0 < nch; q0 += kWave) {
            const int n = min(kWave, nch - q0);
            for (int i = lane; i < n * kStat; i += kWave) s_st[i] = st[(size_t)q0 * kStat + i];
            __syncthreads();
            if (pass == 0)
                pair ? fold_max<true>(s_st, n, ma, ms) : fold_max<false>(s_st, n, ma, ms);
            else
                pair ? fold_sum<true>(s_st, n, ma, ms, za, zs, cross) : fold_sum<false>(s_st, n, ma, ms, za, zs, cross);
            __syncthreads();
        }
    if (lane == 0) {
        write_loss(p, b, ma, ms, za, zs, cross);
        st[0] = ma, st[1] = za, st[3] = ms, st[4] = zs;
    }
}

// Phase 2, bf16: the logit gradients as MFMA operands, without an fp32 copy in memory. Workgroup
// (512 vocabulary entries, rows 8 y .. 8 y + 7), one wave: the rows' statistics combined in chunk
// order (staged through LDS), then each thread forms the gradients of 8 vocabulary entries x 8 rows
// and writes the GEMM operand of dH = D W (rows r < rows, contraction over the vocabulary, Dact: two
// planes of cap rows x ldz) and the operand of dW = D^T H (contraction over the rows, DT: two planes
// of ldz x rpad, rows rows .. rpad - 1 zero). Latency bounds it: every logit load is issued before
// the first is used. At the 7B head
// (64 rows) 20 us in the place of 10 (fp32 gradients) + 12 (their packing) and a launch.
//
// FOLDED: the statistics of a row are already one chunk (loss_fold_kernel). A vocabulary of more than
// kStageChunks chunks takes it: the stage of eight rows is 160 bytes a chunk and every workgroup
// repeats the fold, so from there on (20 KiB, eight workgroups per CU) the stage limits the waves on
// a CU, and above a million entries it would not fit the LDS.
constexpr int kGradThreads = kWave, kStageChunks = 128;
template <bool FOLDED>
__global__ __launch_bounds__(kGradThreads) void loss_grad_pack_kernel(LossParams p, const float *stats, int nch, int cap,
                                                                      uint16_t *Dact, int rpad, uint16_t *DT) {
    struct Row {
        const float *a, *s;  // teacher and student logits (AR row: a only)
        float ma, ia, ms, is;
        int t, kind;         // kind 0: no row, 1: pair, 2: AR row, 3: AR row with a target outside the vocabulary
    };
    __shared__ Row s_row[8];
    extern __shared__ float s_stat[];  // the statistics of the eight rows [8][nch][kStat]
    const int c = blockIdx.x, r0 = blockIdx.y * 8, tid = threadIdx.x, V = p.V, rows = p.P + p.A;
    if constexpr (!FOLDED) {
        for (int i = tid; i < min(8, rows - r0) * nch * kStat; i += kGradThreads)
            s_stat[i] = stats[(size_t)r0 * nch * kStat + i];
        __syncthreads();
    }
    if (tid < 8) {
        Row q{p.Z, p.Z, 0.f, 0.f, 0.f, 0.f, 0, 0};  // no row: loads row 0, uses none of it
        const int b = r0 + tid;
        if (b < rows) {
            const bool pair = b < p.P;
            float ma = -INFINITY, ms = -INFINITY, za = 0.f, zs = 0.f, cross = 0.f;
            if constexpr (FOLDED) {
                const float *st = stats + (size_t)b * nch * kStat;  // where loss_fold_kernel left them
                ma = st[0], za = st[1], ms = st[3], zs = st[4];
            } else {
                const float *st = s_stat + tid * nch * kStat;
                if (pair) {
                    fold_max<true>(st, nch, ma, ms);
                    fold_sum<true>(st, nch, ma, ms, za, zs, cross);
                } else {
                    fold_max<false>(st, nch, ma, ms);
                    fold_sum<false>(st, nch, ma, ms, za, zs, cross);
                }
                if (c == 0) write_loss(p, b, ma, ms, za, zs, cross);
            }
            if (pair) {
                q = Row{p.Z + (size_t)b * p.ldz, p.Z + (size_t)(p.P + b) * p.ldz, ma, 1.0f / za, ms, 1.0f / zs, 0, 1};
            } else {
                const int i = b - p.P, t = p.targets[i];
                const float *z = p.Z + (size_t)(2 * p.P + i) * p.ldz;
                q = Row{z, z, ma, 1.0f / za, 0.f, 0.f, t, t < 0 || t >= V ? 3 : 2};
            }
        }
        s_row[tid] = q;
    }
    __syncthreads();
    const int v0 = (c * kGradThreads + tid) * 8;
    if (v0 >= p.ldz) return;  // ldz is a multiple of 64
    f32x4 za[8][2], zs[8][2];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            za[i][h] = *reinterpret_cast<const f32x4 *>(s_row[i].a + v0 + 4 * h);
            zs[i][h] = *reinterpret_cast<const f32x4 *>(s_row[i].s + v0 + 4 * h);
        }
    float x[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const Row q = s_row[i];  // uniform
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float a = za[i][e >> 2][e & 3], s = zs[i][e >> 2][e & 3];
            float y = 0.f;
            if (q.kind == 1)
                y = expf(s - q.ms) * q.is - expf(a - q.ma) * q.ia;
            else if (q.kind == 2)
                y = p.omega * (expf(a - q.ma) * q.ia - (v0 + e == q.t ? 1.0f : 0.0f));
            else if (q.kind == 3)
                y = NAN;
            x[i][e] = v0 + e < V ? y : 0.f;  // padding columns carry no gradient
        }
    }
    const size_t pa = act_plane(cap, p.ldz), pt = (size_t)p.ldz * rpad;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (r0 + i >= rows) break;
        u32x4 h, l;
        split8(x[i], h, l);
        const size_t o = act_idx<Prec::BF16>(r0 + i, v0, p.ldz);  // 8 consecutive entries: one vector
        *reinterpret_cast<u32x4 *>(Dact + o) = h;
        *reinterpret_cast<u32x4 *>(Dact + pa + o) = l;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        float y[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) y[i] = x[i][j];
        u32x4 h, l;
        split8(y, h, l);
        const size_t o = tr_idx(v0 + j, r0, rpad / 32);
        *reinterpret_cast<u32x4 *>(DT + o) = h;
        *reinterpret_cast<u32x4 *>(DT + pt + o) = l;
    }
}

// fp32: the GEMM operand of dH = D W only (dW takes D as it is).
__global__ void pack_d_f32_kernel(const float *D, int rows, int ldd, int Vp, int cap, float *Dact) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)rows * Vp) return;
    const int r = (int)(i / Vp), v = (int)(i % Vp);
    Dact[act_idx<Prec::F32>(r, v, Vp)] = D[(size_t)r * ldd + v];
}

// The packed LM head W [Vp][d] (tiles over (k-step of d, 16 vocabulary rows)) repacked as W^T
// [d][Vp] (tiles over (k-step of the vocabulary, 16 columns of d)), the weight operand of
// dH = D W. Thread: a VEC x VEC block (VEC vocabulary rows from v0, VEC columns from k0), read as
// VEC vectors along d and written as VEC vectors along the vocabulary.
template <Prec P>
__global__ __launch_bounds__(256) void transpose_lm_kernel(const uint8_t *W, int Vp, int d, uint8_t *WT) {
    using PT = PrecT<P>;
    using T = typename PT::T;
    constexpr int VEC = PT::VEC, KSTEP = PT::KSTEP;
    const int nvb = Vp / VEC;
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int vb = (int)(t % nvb), kb = (int)(t / nvb);
    if (kb >= d / VEC) return;
    const int v0 = vb * VEC, k0 = kb * VEC, Tv = Vp / 16, Td = d / 16;
    T x[VEC][VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        const int v = v0 + i;
        const size_t tile = (size_t)(k0 / KSTEP) * Tv + v / 16;
        const int lane = 16 * ((k0 % KSTEP) / VEC) + v % 16;
        const u32x4 q = *reinterpret_cast<const u32x4 *>(W + tile * kTileBytes + (size_t)lane * 16);
        const T *e = reinterpret_cast<const T *>(&q);
#pragma unroll
        for (int j = 0; j < VEC; ++j) x[i][j] = e[j];
    }
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        const int k = k0 + j;
        const size_t tile = (size_t)(v0 / KSTEP) * Td + k / 16;
        const int lane = 16 * ((v0 % KSTEP) / VEC) + k % 16;
        alignas(16) T y[VEC];
#pragma unroll
        for (int i = 0; i < VEC; ++i) y[i] = x[i][j];
        *reinterpret_cast<u32x4 *>(WT + tile * kTileBytes + (size_t)lane * 16) = *reinterpret_cast<const u32x4 *>(y);
    }
}

// Sum of the K-split partials in split order; rows < np go to dS, the rest to dA. The last
// workgroup forms *loss (if any) = sum kl + omega * sum nll, each sum in row order, in double.
__global__ __launch_bounds__(256) void loss_dh_sum_kernel(const float *part, int nsplit, int n, int np_d, float *dS, float *dA,
                                                          const float *kl, int np, const float *nll, int na, float omega,
                                                          double *loss) {
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;  // rows are a multiple of 64 floats
    if (i >= (size_t)n) {
        if (!loss || blockIdx.x != gridDim.x - 1 || threadIdx.x != 255) return;  // the last workgroup holds no rows
        double ks = 0.0, ns = 0.0;
        for (int r = 0; r < np; ++r) ks += (double)kl[r];
        for (int r = 0; r < na; ++r) ns += (double)nll[r];
        *loss = ks + (double)omega * ns;
        return;
    }
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int c = 0; c < nsplit; ++c) s += *reinterpret_cast<const f32x4 *>(part + (size_t)c * n + i);
    float *out = i < (size_t)np_d ? dS + i : dA + (i - np_d);
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = s[e];  // the caller's arrays: 4-byte alignment is all that is known
}

// One workgroup per row: out = x (.) g / sqrt(mean(x^2) + eps), the LM head's input row.
__global__ __launch_bounds__(kLossThreads) void hidden_rows_kernel(const float *__restrict__ X, int ldx, int d,
                                                                   const float *__restrict__ g, float eps,
                                                                   float *__restrict__ out) {
    __shared__ float s_buf[4];
    const float *x = X + (size_t)blockIdx.x * ldx;
    float ss = 0.f;
    // eight loads in flight per thread (one at a time, 4096 columns took 8.8 us; 4.0 now)
#pragma unroll 8
    for (int k = threadIdx.x; k < d; k += kLossThreads) ss += x[k] * x[k];
    ss = block_reduce<false>(ss, s_buf);
    const float inv = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll 8
    for (int k = threadIdx.x; k < d; k += kLossThreads) out[(size_t)blockIdx.x * d + k] = x[k] * g[k] * inv;
}

// dW = D^T H, bf16 operands (hi + lo planes; the products hi hi + hi lo + lo hi, fp32
// accumulation). Workgroup: 128 vocabulary rows x 128 columns; wave (wv, wk) owns 64 x 64 (4 x 4
// tiles of 16 x 16); the contraction runs over the rpad rows, 32 per k-step. Writing dW bounds it
// (524 MB at the 7B head): the block goes out through LDS in 512-byte row pieces, nontemporal, so
// that the written lines do not displace the operands and dirty the last-level cache for the next
// kernels. At the 7B head, 64 rows, random operands, launches back to back: 108 us (4.9 TB/s) against
// 145 with ordinary stores; 64 x 256 blocks 110; one workgroup per strip of blocks with its H
// operand kept in registers 104, but slower in a whole call (298 against 286 us); 16-byte stores
// straight from the registers (64-byte row pieces) 159.
//
// dW is the caller's, of which 4-byte alignment is all that is known: the store type says so, and the
// hardware takes a 16-byte store at any 4-byte address.
constexpr int kDwV = 128, kDwK = 128, kDwLd = kDwK + 4;  // LDS row stride (floats)
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
__global__ __launch_bounds__(256) void loss_dw_mfma_kernel(const uint16_t *DT, const uint16_t *HT, int Vp, int d,
                                                           int rpad, int V, float *dW) {
    extern __shared__ float s_blk[];  // kDwV x kDwLd
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, wv = w & 1, wk = w >> 1;
    const int nvt = Vp / 16, nkt = d / 16, ks = rpad / 32;
    // grid x: column blocks (fastest, so consecutive workgroups share the block of D^T through
    // L2), y: vocabulary blocks
    const int vt0 = blockIdx.y * (kDwV / 16) + wv * 4, kt0 = blockIdx.x * (kDwK / 16) + wk * 4;
    const size_t pd = (size_t)Vp * rpad, ph = (size_t)d * rpad;
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < ks; ++s) {
        u32x4 ah[4], al[4], bh[4], bl[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int vt = min(vt0 + i, nvt - 1);  // tiles past the end recompute the last (not stored)
            const size_t o = ((size_t)(vt * ks + s) * kWave + lane) * 8;
            ah[i] = *reinterpret_cast<const u32x4 *>(DT + o);
            al[i] = *reinterpret_cast<const u32x4 *>(DT + pd + o);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int kt = min(kt0 + j, nkt - 1);
            const size_t o = ((size_t)(kt * ks + s) * kWave + lane) * 8;
            bh[j] = *reinterpret_cast<const u32x4 *>(HT + o);
            bl[j] = *reinterpret_cast<const u32x4 *>(HT + ph + o);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[i][j] = mfma_kstep<Prec::BF16>(ah[i], bh[j], acc[i][j]);
                acc[i][j] = mfma_kstep<Prec::BF16>(ah[i], bl[j], acc[i][j]);
                acc[i][j] = mfma_kstep<Prec::BF16>(al[i], bh[j], acc[i][j]);
            }
    }
    // C layout: row 4 * (lane / 16) + e of tile (i, j), column lane % 16
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                s_blk[(64 * wv + 16 * i + 4 * (lane >> 4) + e) * kDwLd + 64 * wk + 16 * j + (lane & 15)] = acc[i][j][e];
    __syncthreads();
    // two rows of the block per store: 32 lanes of 16 bytes each
    const int c = 4 * (lane & 31), k = blockIdx.x * kDwK + c;
    if (k < d) {
#pragma unroll 4
        for (int r = 2 * w + (lane >> 5); r < kDwV; r += 8) {
            const int v = kDwV * blockIdx.y + r;
            if (v < V)
                __builtin_nontemporal_store(*reinterpret_cast<const f32x4 *>(s_blk + r * kDwLd + c),
                                            reinterpret_cast<f32x4_a4 *>(dW + (size_t)v * d + k));
        }
    }
}

// dW, fp32 operands: workgroup (64 vocabulary rows, 64 columns of d); wave w owns rows
// 16w..16w+15 and the 64 columns (four 16-column tiles); the sum runs over the gradient rows,
// 4 at a time.
__global__ __launch_bounds__(256) void loss_dw_f32_kernel(const float *D, int rows, int ldd, const float *S0, int np,
                                                          const float *R0, int d, int V, float *dW) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int v = blockIdx.x * 64 + 16 * w + (lane & 15), kb = blockIdx.y * 64;
    f32x4 acc[4];
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) acc[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int r0 = 0; r0 < rows; r0 += 4) {
        const int r = r0 + (lane >> 4);
        const float a = (r < rows && v < V) ? D[(size_t)r * ldd + v] : 0.f;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
            const int k = kb + 16 * kt + (lane & 15);
            const float b = r >= rows ? 0.f : r < np ? S0[(size_t)r * d + k] : R0[(size_t)(r - np) * d + k];
            acc[kt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[kt], 0, 0, 0);
        }
    }
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int vo = blockIdx.x * 64 + 16 * w + 4 * (lane >> 4) + j;
            if (vo < V) dW[(size_t)vo * d + kb + 16 * kt + (lane & 15)] = acc[kt][j];
        }
}

static bool loss_params_ok(const LossParams &p) { return p.P >= 0 && p.A >= 0 && p.P + p.A >= 1 && p.V >= 1 && p.ldz >= p.V; }

hipError_t launch_loss_stats(const LossParams &p, float *stats, hipStream_t s, hipEvent_t e0) {
    if (!loss_params_ok(p)) return hipErrorInvalidValue;
    const int nch = (p.ldz + kLossChunk - 1) / kLossChunk;  // = chunks of V (ldz - V < 64 <= kLossChunk)
    hipExtLaunchKernelGGL(loss_stats_kernel, dim3(nch, p.P + p.A), dim3(kLossThreads), 0, s, e0, nullptr, 0, p, stats, nch);
    return hipGetLastError();
}

hipError_t launch_loss_grad_f32(const LossParams &p, const float *stats, int cap, float *Dact, hipStream_t s, hipEvent_t e1) {
    const int rows = p.P + p.A;
    if (!loss_params_ok(p) || rows > cap) return hipErrorInvalidValue;
    const int nch = (p.ldz + kLossChunk - 1) / kLossChunk;
    hipLaunchKernelGGL(loss_grad_kernel, dim3(nch, rows), dim3(kLossThreads), 0, s, p, stats, nch);
    const size_t n = (size_t)rows * p.ldz;
    hipExtLaunchKernelGGL(pack_d_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, nullptr, e1, 0,
                          (const float *)p.D, rows, p.ldz, p.ldz, cap, Dact);
    return hipGetLastError();
}

hipError_t launch_loss_grad_pack(const LossParams &p, float *stats, int cap, uint16_t *Dact, int rpad, uint16_t *DT,
                                 hipStream_t s, hipEvent_t e1) {
    const int rows = p.P + p.A;
    if (!loss_params_ok(p) || rows > cap || p.ldz % 64 != 0 || rpad % 32 != 0 || rpad < rows) return hipErrorInvalidValue;
    const int nch = (p.ldz + kLossChunk - 1) / kLossChunk;
    const dim3 grid((p.ldz / 8 + kGradThreads - 1) / kGradThreads, rpad / 8), block(kGradThreads);
    if (nch > kStageChunks) {
        hipLaunchKernelGGL(loss_fold_kernel, dim3(rows), dim3(kWave), 0, s, p, stats, nch);
        hipExtLaunchKernelGGL(loss_grad_pack_kernel<true>, grid, block, 0, s, nullptr, e1, 0, p, (const float *)stats, nch,
                              cap, Dact, rpad, DT);
    } else {
        hipExtLaunchKernelGGL(loss_grad_pack_kernel<false>, grid, block, (size_t)8 * nch * kStat * sizeof(float), s,
                              nullptr, e1, 0, p, (const float *)stats, nch, cap, Dact, rpad, DT);
    }
    return hipGetLastError();
}

hipError_t launch_pack_inputs(bool bf16, const float *T0, const float *S0, int np, const float *R0, int na, int d, int cap,
                              void *A, int rpad, uint16_t *HT, hipStream_t s, hipEvent_t e0) {
    const int rows = 2 * np + na;
    if (np < 0 || na < 0 || rows < 1 || rows > cap || d % 64 != 0) return hipErrorInvalidValue;
    if (!bf16) {
        const size_t n = (size_t)rows * d;
        hipExtLaunchKernelGGL(pack_rows_kernel<Prec::F32>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, e0, nullptr,
                              0, T0, S0, np, R0, na, d, cap, A);
        return hipGetLastError();
    }
    if (rpad % 32 != 0 || rpad < np + na) return hipErrorInvalidValue;
    const int n_rows = (rows * (d / 8) + 255) / 256, n_ht = (d * (rpad / 8) + 255) / 256;
    hipExtLaunchKernelGGL(pack_inputs_kernel, dim3(n_rows + n_ht), dim3(256), 0, s, e0, nullptr, 0, T0, S0, np, R0, na, d,
                          cap, reinterpret_cast<uint16_t *>(A), n_rows, rpad, HT);
    return hipGetLastError();
}

hipError_t launch_transpose_lm(bool bf16, const uint8_t *W, int Vp, int d, uint8_t *WT, hipStream_t s) {
    if (Vp % 64 != 0 || d % 64 != 0) return hipErrorInvalidValue;
    const int vec = bf16 ? PrecT<Prec::BF16>::VEC : PrecT<Prec::F32>::VEC;
    const size_t n = (size_t)(Vp / vec) * (d / vec);
    const dim3 grid((unsigned)((n + 255) / 256));
    if (bf16)
        hipLaunchKernelGGL(transpose_lm_kernel<Prec::BF16>, grid, dim3(256), 0, s, W, Vp, d, WT);
    else
        hipLaunchKernelGGL(transpose_lm_kernel<Prec::F32>, grid, dim3(256), 0, s, W, Vp, d, WT);
    return hipGetLastError();
}

hipError_t launch_loss_dh_sum(const float *part, int nsplit, int rows, int d, const LossParams &p, float *dS, float *dA,
                              double *loss, hipStream_t s, hipEvent_t e1) {
    if (nsplit < 1 || rows < 1 || p.P < 0 || p.P > rows || d % 64 != 0) return hipErrorInvalidValue;
    const int n = rows * d;
    hipExtLaunchKernelGGL(loss_dh_sum_kernel, dim3((n / 4 + 255) / 256 + 1), dim3(256), 0, s, nullptr, e1, 0, part, nsplit, n,
                          p.P * d, dS, dA, (const float *)p.kl, p.P, (const float *)p.nll, p.A, p.omega, loss);
    return hipGetLastError();
}

hipError_t launch_hidden_rows(const float *X, int ldx, int rows, int d, const float *g, float eps, float *out,
                              hipStream_t s) {
    if (rows < 1 || d < 1 || ldx < d) return hipErrorInvalidValue;
    hipLaunchKernelGGL(hidden_rows_kernel, dim3(rows), dim3(kLossThreads), 0, s, X, ldx, d, g, eps, out);
    return hipGetLastError();
}

hipError_t launch_loss_dw(bool bf16, const uint16_t *DT, const uint16_t *HT, int Vp, int rpad, const float *D,
                          int rows, int ldd, const float *S0, int np, const float *R0, int d, int V, float *dW,
                          hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    if (rows < 1 || rows > 64 || np < 0 || np > rows || d % 64 != 0 || ldd < V || Vp < V || Vp % 64 != 0)
        return hipErrorInvalidValue;
    if (bf16) {
        if (rpad % 32 != 0 || rpad < rows) return hipErrorInvalidValue;
        const dim3 grid((d + kDwK - 1) / kDwK, (Vp + kDwV - 1) / kDwV);
        const size_t lds = (size_t)kDwV * kDwLd * sizeof(float);
        if (e0)
            hipExtLaunchKernelGGL(loss_dw_mfma_kernel, grid, dim3(256), lds, s, e0, e1, 0, DT, HT, Vp, d, rpad, V, dW);
        else
            hipLaunchKernelGGL(loss_dw_mfma_kernel, grid, dim3(256), lds, s, DT, HT, Vp, d, rpad, V, dW);
        return hipGetLastError();
    }
    const dim3 grid((V + 63) / 64, d / 64);
    if (e0)
        hipExtLaunchKernelGGL(loss_dw_f32_kernel, grid, dim3(256), 0, s, e0, e1, 0, D, rows, ldd, S0, np, R0, d, V, dW);
    else
        hipLaunchKernelGGL(loss_dw_f32_kernel, grid, dim3(256), 0, s, D, rows, ldd, S0, np, R0, d, V, dW);
    return hipGetLastError();
}

}  // namespace cllm
