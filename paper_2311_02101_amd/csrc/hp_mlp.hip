// Learned initial assignments: per-variable features, a 32 -> 256 -> 1
// perceptron (bfloat16 weights on MFMA, FP32 accumulation) with its training
// kernels (backward with the forward recomputed, a fixed-order reduction of
// its partial sums, Adam), and the initial Bernoulli draws.
//
// Features (per variable, exact dyadic values before one bfloat16 rounding):
//   0..13  clauses of real length l = 1..7 holding the variable positively
//          (index 2(l-1)) / negated (2(l-1)+1), divided by 8
//   14, 15 positive / negated occurrences / 8;  16 their difference / 8
//   17, 18 sum over positive / negated occurrences of 2^-l;  19 difference
//   20..31 zero
// The real length ignores the trailing padding copies of a clause's first
// literal.  Network: q = sigmoid(w2 . relu(W1^T x + b1) + b2).
#include <hip/hip_runtime.h>

#include <cmath>

#include "hp_internal.hpp"
#include "philox.hpp"

namespace hp {

constexpr int kF = HP_MLP_IN;
constexpr int kH = HP_MLP_HIDDEN;
constexpr int kOffW1 = 0, kOffB1 = kF * kH, kOffW2 = kOffB1 + kH, kOffB2 = kOffW2 + kH;

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;

__device__ __forceinline__ uint16_t bf16_bits(float x) {
    const __bf16 b = (__bf16)x;   // round to nearest even
    return __builtin_bit_cast(uint16_t, b);
}
__device__ __forceinline__ float bf16_value(uint16_t u) {
    return __builtin_bit_cast(float, (uint32_t)u << 16);
}

// ---- features ----------------------------------------------------------------
// One workgroup per tile of 1024 variables: it scans the formula's clause
// records and counts, in LDS, the 14 (length, sign) occurrences of its
// variables; every other feature is a sum of those counts.  Bound by the LDS
// counter updates and the scan (16 bytes a clause and tile, from L2 after the
// formula's first tile).  Three FP32 global atomics per literal took, before, at
// about 20 G atomics/s: 16 formulas of 2000 variables and 12 000 clauses 207 -> 12
// us, one of 30 000 and 100 000 111 -> 55 us.  A formula has as many workgroups as
// tiles: one of 64 variables and 30 000 clauses runs on one CU (193 -> 20 us).
// 57 KB of counters let two workgroups of 1024 threads share a CU.
constexpr int kFeatThreads = 1024;
constexpr int kFeatBins = 14;

__global__ __launch_bounds__(kFeatThreads) void feature_kernel(const uint4 *__restrict__ rec,
                                                               const FormulaDev *__restrict__ fd,
                                                               const VarTile *__restrict__ tile,
                                                               uint16_t *__restrict__ x, bool vec) {
    __shared__ uint32_t s_cnt[kFeatBins][kTileVars];
    const VarTile t = tile[blockIdx.x];
    const FormulaDev &f = fd[t.f];
    const uint4 *__restrict__ r = rec + f.clause_off;
    const int C = f.c, nv = min(kTileVars, f.n - t.i0), tid = threadIdx.x;
    for (int i = tid; i < kFeatBins * kTileVars; i += kFeatThreads) (&s_cnt[0][0])[i] = 0u;
    __syncthreads();
    auto count = [&](const uint4 &q) {
        const uint32_t e[7] = {q.x & 0xffffu, q.x >> 16, q.y & 0xffffu, q.y >> 16, q.z & 0xffffu, q.z >> 16,
                               q.w & 0xffffu};
        const int len = (int)rec_len(q.w);
#pragma unroll
        for (int k = 0; k < kMaxK; ++k) {
            if (k < len) {
                const uint32_t i = (e[k] & 0x7fffu) - (uint32_t)t.i0;
                if (i < (uint32_t)nv) atomicAdd(&s_cnt[2 * (len - 1) + (int)(e[k] >> 15)][i], 1u);
            }
        }
    };
    // two records in flight per thread
    int c = tid;
    for (; c + kFeatThreads < C; c += 2 * kFeatThreads) {
        const uint4 q0 = r[c], q1 = r[c + kFeatThreads];
        count(q0);
        count(q1);
    }
    if (c < C) count(r[c]);
    __syncthreads();
    // four threads write the 64-byte row of a variable, 16 bytes (8 features) each
    uint16_t *__restrict__ row = x + (size_t)(f.var_off + t.i0) * kF;
    for (int j = tid; j < 4 * nv; j += kFeatThreads) {
        const int i = j >> 2, part = j & 3;
        float g[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        if (part < 3) {
            float cf[kFeatBins];
            uint32_t occ[2] = {0u, 0u};
            double w[2] = {0.0, 0.0};       // sums of 2^-length, exact
#pragma unroll
            for (int b = 0; b < kFeatBins; ++b) {
                const uint32_t n = s_cnt[b][i];
                cf[b] = (float)n * 0.125f;
                occ[b & 1] += n;
                w[b & 1] += (double)n * (1.0 / (double)(2 << (b >> 1)));
            }
            const float p = (float)occ[0], m = (float)occ[1], wp = (float)w[0], wm = (float)w[1];
            if (part == 0) {
#pragma unroll
                for (int b = 0; b < 8; ++b) g[b] = cf[b];
            } else if (part == 1) {
#pragma unroll
                for (int b = 8; b < kFeatBins; ++b) g[b - 8] = cf[b];
                g[6] = p * 0.125f;
                g[7] = m * 0.125f;
            } else {
                g[0] = (p - m) * 0.125f;
                g[1] = wp;
                g[2] = wm;
                g[3] = wp - wm;
            }
        }
        uint32_t o[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) o[b] = (uint32_t)bf16_bits(g[2 * b]) | ((uint32_t)bf16_bits(g[2 * b + 1]) << 16);
        uint16_t *dst = row + (size_t)i * kF + part * 8;
        if (vec) {
            *reinterpret_cast<uint4 *>(dst) = make_uint4(o[0], o[1], o[2], o[3]);
        } else {
#pragma unroll
            for (int b = 0; b < 8; ++b) dst[b] = (uint16_t)(o[b >> 1] >> (16 * (b & 1)));
        }
    }
}

// ---- perceptron ---------------------------------------------------------------
// Hidden layer on MFMA 32x32x16 bf16.  Lane l supplies index l%32 of an operand
// (a row of A, a column of B) with k = (l/32)*8 + 0..7; D[32 x 32]: register
// i -> row (i/4)*8 + (l/32)*4 + i%4, column l%32.  A tile is 32 data rows (A)
// against a chunk of 32 hidden units (B): a lane holds 16 rows of one unit.
//
// Order of a row's output sum, fixed (the initial draws compare 24-bit uniforms
// with q, so another order of the same sum flips one draw in 80 million): unit
// position p = l%32 sums relu(pre) w2 over the eight chunks in ascending order
// (one fused multiply-add each, the bias added to the product before relu), then
// the 32 positions are added as a balanced tree over the bits of p, lowest bit
// first, and b2 last; all in FP32.
constexpr int kStepRows = 128;   // data rows per step of the backward kernel: 4 tiles
constexpr int kChunks = kH / 32;
constexpr int kWStride = 40;     // halves per staged unit: 16-byte aligned, off the banks' period

// row of D register i for lane half h (see above)
__device__ __forceinline__ int d_row(int i, int h) { return (i / 4) * 8 + h * 4 + (i % 4); }

// The network in LDS: W1 transposed ([unit][feature], bfloat16), (b1, w2) per unit.
struct NetLds {
    __align__(16) uint16_t w1t[kH * kWStride];
    float2 bw[kH];
};

__device__ __forceinline__ void load_net(NetLds &s, const float *params, const uint16_t *wbf, int tid, int NT) {
    for (int i = tid; i < kH * kF; i += NT) s.w1t[(i / kF) * kWStride + i % kF] = wbf[i];
    for (int i = tid; i < kH; i += NT) s.bw[i] = make_float2(params[kOffB1 + i], bf16_value(wbf[kH * kF + i]));
}

// this lane's two B operands (k-steps) of chunk j
__device__ __forceinline__ void chunk_weights(const NetLds &s, int j, int lane, bf16x8 &w0, bf16x8 &w1) {
    const uint16_t *w = &s.w1t[(j * 32 + (lane & 31)) * kWStride + (lane >> 5) * 8];
    w0 = *reinterpret_cast<const bf16x8 *>(w);
    w1 = *reinterpret_cast<const bf16x8 *>(w + 16);
}

// The two operands (k-steps) of the 32-row tile starting at row0: lane l
// takes row row0 + l%32, features (l/32)*8 + 0..7 and 16 + (l/32)*8 + 0..7
// (zeros past the last row).  Operands move as integer words: element m of a
// bfloat16 vector is bits 16*(m%2) of word m/2.
__device__ __forceinline__ void load_x_tile(const uint16_t *x, int64_t rows, int64_t row0, int lane, uint4 &x0,
                                            uint4 &x1) {
    const int64_t r = row0 + (lane & 31);
    const int half = lane >> 5;
    x0 = make_uint4(0, 0, 0, 0);
    x1 = make_uint4(0, 0, 0, 0);
    if (r < rows) {
        x0 = *reinterpret_cast<const uint4 *>(x + r * kF + half * 8);
        x1 = *reinterpret_cast<const uint4 *>(x + r * kF + 16 + half * 8);
    }
}

// the value of x in the lane that a VALU lane permute names
template <int kCtrl>
__device__ __forceinline__ float dpp(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), kCtrl, 0xf, 0xf, false));
}

// One level of the tree: of the 2 N sums the lane keeps N (the upper half if
// `hi`) and adds the partner's, whose other half it sends in turn.
template <int N, int kCtrl>
__device__ __forceinline__ void tree_level(float (&s)[16], bool hi) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float keep = hi ? s[i + N] : s[i], send = hi ? s[i] : s[i + N];
        s[i] = keep + dpp<kCtrl>(send);
    }
}

// D register whose row a lane holds after the tree.  The third level pairs
// lanes l and 7 - l of every 8 (a mirror; there is no permute by 4), so in the
// upper four the first two levels keep the opposite halves.
__device__ __forceinline__ int tree_reg(int lane) {
    const int q = (lane & 4) ? ~lane : lane;
    return (q & 1) * 8 + (q & 2) * 2 + (lane >> 1 & 2) + (lane >> 3 & 1);
}

// Output logit (without b2) of row d_row(tree_reg(lane), lane / 32) of the tile,
// the same in lanes l and l ^ 16.  Each level of the tree halves what a lane
// holds (47 VALU instructions a tile, where a sum of every register in every
// lane takes 80 lane permutes and adds).
__device__ __forceinline__ float tile_logit(const NetLds &net, int lane, bf16x8 a0, bf16x8 a1) {
    float s[16] = {};
#pragma unroll 2
    for (int j = 0; j < kChunks; ++j) {
        bf16x8 w0, w1;
        chunk_weights(net, j, lane, w0, w1);
        f32x16 acc = {};
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, w0, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, w1, acc, 0, 0, 0);
        const float2 bw = net.bw[j * 32 + (lane & 31)];
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = fmaf(fmaxf(acc[i] + bw.x, 0.0f), bw.y, s[i]);
    }
    const int q = (lane & 4) ? ~lane : lane;
    tree_level<8, 0xB1>(s, (q & 1) != 0);        // quad_perm 1,0,3,2
    tree_level<4, 0x4E>(s, (q & 2) != 0);        // quad_perm 2,3,0,1
    tree_level<2, 0x141>(s, (lane & 4) != 0);    // row_half_mirror
    tree_level<1, 0x128>(s, (lane & 8) != 0);    // row_ror:8
    return s[0] + __shfl_xor(s[0], 16, kWave);
}

// Forward: a wave per tile.  Bound by the three VALU instructions per row and
// unit that the order asks for: 524 288 rows take 21.4 us, 4 M rows 150 us (460
// TFLOP/s of products); with every register summed over the lanes in every lane
// 37.2 and 245 us; with the weights as A and other sums (bias in the product,
// FP64 over the chunks) 24.6 and 172 us.
constexpr int kFwdWaves = 4;

__global__ __launch_bounds__(kFwdWaves *kWave) void mlp_forward_kernel(const uint16_t *__restrict__ x, int64_t rows,
                                                                       const float *__restrict__ params,
                                                                       const uint16_t *__restrict__ wbf,
                                                                       float *__restrict__ q_out) {
    __shared__ NetLds s_net;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    load_net(s_net, params, wbf, tid, kFwdWaves * kWave);
    __syncthreads();
    const float b2 = params[kOffB2];
    const int row = d_row(tree_reg(lane), lane >> 5);
    const int64_t n_tiles = (rows + 31) / 32;
    for (int64_t tile = (int64_t)blockIdx.x * kFwdWaves + wave; tile < n_tiles; tile += (int64_t)gridDim.x * kFwdWaves) {
        uint4 x0, x1;
        load_x_tile(x, rows, tile * 32, lane, x0, x1);
        const float o = tile_logit(s_net, lane, __builtin_bit_cast(bf16x8, x0), __builtin_bit_cast(bf16x8, x1)) + b2;
        const int64_t r = tile * 32 + row;
        if ((lane & 16) == 0 && r < rows) q_out[r] = 1.0f / (1.0f + expf(-o));
    }
}

// Backward: 8 waves, 128 rows (4 tiles) per step.
//   pass 1: waves 0..3 take a tile each: logits as in the forward kernel, then q,
//           the output gradient g = (q - y) / rows and the loss of the row that a
//           lane holds; waves 4..7 bring the tiles' rows to LDS, as they are and
//           transposed;
//   pass 2: every wave, for its own 32 hidden units: with the rows as A and the
//           units' weights as B, a lane holds 16 rows of its unit: dh = g w2
//           relu'(pre) (bfloat16 for the product) adds x^T dh to the wave's dW1
//           chunk, g h to dw2 and dh to db1.
// The x^T dh product reuses the D layout as its B operand by ordering the
// reduction index (the rows) as D does:
// step s, k = (l/32)*8 + m  <->  row ((s*8 + m)/4)*8 + (l/32)*4 + m%4.
// Each dW1 column is summed by one wave only; a workgroup writes its sums to its
// row of the workspace.  One barrier per step: rows and g have two buffers.
// 262 144 rows take 45.6 us with the reduction below (36.8 and 8.6 under the
// profiler), 4 M rows 384 us; before 93.1 and 1019 us (4 waves, all of them on
// logits with the lane sums, weights from LDS in pass 2 too).  512 workgroups,
// half the rows to reduce, would save 3.5 us of 45.6 but sum twice as many rows in
// a row in FP32.
constexpr int kBwdWaves = 8;
constexpr int kXStride = 40;      // halves per staged row: 16-byte aligned, off the banks' period
constexpr int kXtStride = 36;     // halves per staged feature: 8-byte aligned

__global__ __launch_bounds__(kBwdWaves *kWave) __attribute__((amdgpu_waves_per_eu(4))) void mlp_backward_kernel(
    const uint16_t *__restrict__ x, const float *__restrict__ y, int64_t rows, const float *__restrict__ params,
    const uint16_t *__restrict__ wbf, float *__restrict__ part) {
    __shared__ NetLds s_net;
    __shared__ __align__(16) uint16_t s_x[2][4][32 * kXStride];       // tile rows: [row][feature]
    __shared__ __align__(16) uint16_t s_xt[2][4][kF * kXtStride];     // transposed: [feature][row]
    __shared__ __align__(16) float s_g[2][kStepRows];
    __shared__ float s_red[4][2];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int half = lane >> 5, col_in = lane & 31, col = wave * 32 + col_in;
    load_net(s_net, params, wbf, tid, kBwdWaves * kWave);
    __syncthreads();
    bf16x8 w0, w1;
    chunk_weights(s_net, wave, lane, w0, w1);
    const float b2 = params[kOffB2], bb = s_net.bw[col].x, ww = s_net.bw[col].y;
    const float inv_rows = 1.0f / (float)rows;
    const int row_in = d_row(tree_reg(lane), half);
    const int64_t n_steps = (rows + kStepRows - 1) / kStepRows;
    f32x16 dw1 = {};
    float dw2 = 0.0f, db1 = 0.0f, db2 = 0.0f, lsum = 0.0f;      // db2, lsum: the lane's row in each of its tiles
    int buf = 0;
    for (int64_t step = blockIdx.x; step < n_steps; step += gridDim.x, buf ^= 1) {   // uniform over the workgroup
        // ---- pass 1 ----
        const int tile = wave & 3;
        const int64_t row0 = step * kStepRows + 32 * tile;
        uint4 x0, x1;
        load_x_tile(x, rows, row0, lane, x0, x1);
        if (wave < 4) {
            const float o =
                tile_logit(s_net, lane, __builtin_bit_cast(bf16x8, x0), __builtin_bit_cast(bf16x8, x1)) + b2;
            if ((lane & 16) == 0) {
                const int64_t r = row0 + row_in;
                float g = 0.0f;
                if (r < rows) {
                    const float yy = y[r];
                    const float qq = 1.0f / (1.0f + expf(-o));
                    g = (qq - yy) * inv_rows;
                    // softplus(o) - y o
                    const float sp = o > 0.0f ? o + log1pf(expf(-o)) : log1pf(expf(o));
                    lsum += sp - yy * o;
                    db2 += g;
                }
                s_g[buf][32 * tile + row_in] = g;
            }
        } else {
            uint16_t *xr = &s_x[buf][tile][col_in * kXStride + half * 8];
            *reinterpret_cast<uint4 *>(xr) = x0;
            *reinterpret_cast<uint4 *>(xr + 16) = x1;
            const uint32_t v0[4] = {x0.x, x0.y, x0.z, x0.w}, v1[4] = {x1.x, x1.y, x1.z, x1.w};
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                s_xt[buf][tile][(half * 8 + m) * kXtStride + col_in] = (uint16_t)(v0[m >> 1] >> (16 * (m & 1)));
                s_xt[buf][tile][(16 + half * 8 + m) * kXtStride + col_in] = (uint16_t)(v1[m >> 1] >> (16 * (m & 1)));
            }
        }
        // (the next step's pass 1 writes the other buffers, whose readers have
        // passed this barrier)
        __syncthreads();
        // ---- pass 2: the wave's units over the 4 tiles ----
#pragma unroll 1
        for (int t = 0; t < 4; ++t) {
            const uint16_t *xr = &s_x[buf][t][col_in * kXStride + half * 8];
            const bf16x8 a0 = *reinterpret_cast<const bf16x8 *>(xr);
            const bf16x8 a1 = *reinterpret_cast<const bf16x8 *>(xr + 16);
            // x^T with rows in the D-register order: 4 consecutive rows a read
            const uint16_t *xt = &s_xt[buf][t][col_in * kXtStride + half * 4];
            uint2 p[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) p[m] = *reinterpret_cast<const uint2 *>(xt + 8 * m);
            const bf16x8 ax0 = __builtin_bit_cast(bf16x8, make_uint4(p[0].x, p[0].y, p[1].x, p[1].y));
            const bf16x8 ax1 = __builtin_bit_cast(bf16x8, make_uint4(p[2].x, p[2].y, p[3].x, p[3].y));
            f32x16 acc = {};
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, w0, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, w1, acc, 0, 0, 0);
            uint32_t dq[8];
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const float4 g4 = *reinterpret_cast<const float4 *>(&s_g[buf][32 * t + q4 * 8 + half * 4]);
                const float g[4] = {g4.x, g4.y, g4.z, g4.w};
                float dh[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float pre = acc[4 * q4 + k] + bb;
                    dw2 = fmaf(g[k], fmaxf(pre, 0.0f), dw2);
                    dh[k] = pre > 0.0f ? g[k] * ww : 0.0f;
                    db1 += dh[k];
                }
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    dq[2 * q4 + k] = __builtin_bit_cast(
                        uint32_t, __builtin_convertvector((f32x2){dh[2 * k], dh[2 * k + 1]}, bf16x2));
            }
            const bf16x8 d0 = __builtin_bit_cast(bf16x8, make_uint4(dq[0], dq[1], dq[2], dq[3]));
            const bf16x8 d1 = __builtin_bit_cast(bf16x8, make_uint4(dq[4], dq[5], dq[6], dq[7]));
            dw1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ax0, d0, dw1, 0, 0, 0);
            dw1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ax1, d1, dw1, 0, 0, 0);
        }
    }
    // ---- the workgroup's row of the workspace (plain stores) ----
    float *row = part + (size_t)blockIdx.x * (HP_MLP_PARAMS + 1);
#pragma unroll
    for (int i = 0; i < 16; ++i) row[kOffW1 + d_row(i, half) * kH + col] = dw1[i];
    // both halves of the wave hold partials of column col
    const float w2s = dw2 + __shfl_xor(dw2, 32, kWave);
    const float b1s = db1 + __shfl_xor(db1, 32, kWave);
    if (half == 0) {
        row[kOffW2 + col] = w2s;
        row[kOffB1 + col] = b1s;
    }
    // b2 and the loss: a balanced tree over a tile's rows, lowest bit of the row
    // first (the lanes that differ in it: see tree_reg), then the tiles in order
    if (wave < 4) {
        for (int off : {8, 7, 32, 2, 1}) {
            db2 += __shfl_xor(db2, off, kWave);
            lsum += __shfl_xor(lsum, off, kWave);
        }
        if (lane == 0) {
            s_red[wave][0] = db2;
            s_red[wave][1] = lsum;
        }
    }
    __syncthreads();
    if (tid == 0) {
        row[kOffB2] = ((s_red[0][0] + s_red[1][0]) + s_red[2][0]) + s_red[3][0];
        row[HP_MLP_PARAMS] = ((s_red[0][1] + s_red[1][1]) + s_red[2][1]) + s_red[3][1];
    }
}

// grad[p] (p < HP_MLP_PARAMS) and the loss (p = HP_MLP_PARAMS) = the sum of
// column p over the workspace's first `parts` rows, in a fixed order: 16 row
// groups per column summed by 16 waves, then the groups in order.  A wave
// reads 64 consecutive columns of a row (256 bytes) per load.
__global__ __launch_bounds__(1024) void mlp_reduce_kernel(const float *__restrict__ part, int parts,
                                                          float *__restrict__ grad, float *__restrict__ loss_sum) {
    __shared__ float s[16][64];
    const int c = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + c;
    const int per = (parts + 15) / 16, lo = grp * per, hi = min(parts, lo + per);
    float sum = 0.0f;
    if (p <= HP_MLP_PARAMS)
#pragma unroll 8
        for (int b = lo; b < hi; ++b) sum += part[(size_t)b * (HP_MLP_PARAMS + 1) + p];
    s[grp][c] = sum;
    __syncthreads();
    if (grp == 0 && p <= HP_MLP_PARAMS) {
        float t = s[0][c];
        for (int k = 1; k < 16; ++k) t += s[k][c];
        if (p < HP_MLP_PARAMS) grad[p] = t;
        else *loss_sum = t;
    }
}

// ---- Adam and the bfloat16 weight copies --------------------------------------
__global__ void adam_kernel(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                            const float *__restrict__ g, float lr, float beta1, float beta2, float eps,
                            float corr1, float corr2, uint16_t *__restrict__ wbf) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= HP_MLP_PARAMS) return;
    const float gi = g[i];
    const float mi = beta1 * m[i] + (1.0f - beta1) * gi;
    const float vi = beta2 * v[i] + (1.0f - beta2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / corr1) / (sqrtf(vi / corr2) + eps);
    p[i] = pi;
    if (i < kOffB1) {
        const int f = i / kH, col = i % kH;
        wbf[col * kF + f] = bf16_bits(pi);
    } else if (i >= kOffW2 && i < kOffB2) {
        wbf[kH * kF + (i - kOffW2)] = bf16_bits(pi);
    }
}

__global__ void weights_to_bf16_kernel(const float *__restrict__ p, uint16_t *__restrict__ wbf) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kOffB1) {
        const int f = i / kH, col = i % kH;
        wbf[col * kF + f] = bf16_bits(p[i]);
    } else if (i >= kOffW2 && i < kOffB2) {
        wbf[kH * kF + (i - kOffW2)] = bf16_bits(p[i]);
    }
}

// Four consecutive bytes at any alignment (the rows of a state start wherever
// the formula's size puts them), the first m of them if fewer are left.
__device__ __forceinline__ uint32_t load_bytes4(const uint8_t *p, int m) {
    uint32_t w = 0;
    if (m >= 4) {
        __builtin_memcpy(&w, p, 4);
    } else {
        for (int k = 0; k < m; ++k) w |= (uint32_t)p[k] << (8 * k);
    }
    return w;
}
__device__ __forceinline__ void store_bytes4(uint8_t *p, uint32_t w, int m) {
    if (m >= 4) {
        __builtin_memcpy(p, &w, 4);
    } else {
        for (int k = 0; k < m; ++k) p[k] = (uint8_t)(w >> (8 * k));
    }
}

// ---- initial assignments v = [U < q] at the reserved time 2^64 - 1 -------------
// A thread owns one group of four variables (the words of one Philox block)
// of a tile and walks over the chains: the block is evaluated once for its
// four variables, q stays in registers and a chain's four bytes are one
// store.  Bound by the generator (about 60 lane instructions per four variables
// and chain): 32 chains of 256 formulas of 2048 variables take 12.9 us, before
// 88 us with a block, a search for the formula and a byte store per variable.
constexpr int kTileGroups = kTileVars / 4;

__global__ __launch_bounds__(kTileGroups) void init_chains_kernel(const float *__restrict__ q,
                                                                  const FormulaDev *__restrict__ fd,
                                                                  const VarTile *__restrict__ tile, int B, int lo,
                                                                  int hi, uint32_t key0, uint32_t key1,
                                                                  uint8_t *__restrict__ v) {
    const VarTile t = tile[blockIdx.x];
    const int n = fd[t.f].n;
    const int64_t off = fd[t.f].var_off;
    const int i = t.i0 + 4 * (int)threadIdx.x, m = n - i;
    if (m <= 0) return;
    float qv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) qv[k] = k < m ? q[off + i + k] : 0.0f;
    const Key2 key{key0, key1 ^ (uint32_t)t.f};
    for (int b = lo + (int)blockIdx.y; b < hi; b += (int)gridDim.y) {
        const uint4 r = philox4x32_10(make_uint4(0xffffffffu, (uint32_t)b, kPhaseVisible | (uint32_t)(i >> 2),
                                                 0xffffffffu), key);
        const uint32_t rw[4] = {r.x, r.y, r.z, r.w};
        uint32_t w = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float u = (float)(rw[k] >> 8) * (1.0f / 16777216.0f);
            w |= (u < qv[k] ? 1u : 0u) << (8 * k);
        }
        store_bytes4(v + off * B + (int64_t)b * n + i, w, m);
    }
}

// ---- per-variable mean over the chains of a state-layout byte array -------------
// A thread sums four variables over the chains, one four-byte load per chain:
// 5.3 us for 32 chains of 128 formulas of 2048 variables (8.4 MB), before 12.1 us
// with a byte load per variable and a search for the formula.
__global__ __launch_bounds__(kTileGroups) void chain_mean_kernel(const uint8_t *__restrict__ a,
                                                                 const FormulaDev *__restrict__ fd,
                                                                 const VarTile *__restrict__ tile, int B,
                                                                 float *__restrict__ out) {
    const VarTile t = tile[blockIdx.x];
    const int n = fd[t.f].n;
    const int64_t off = fd[t.f].var_off;
    const int i = t.i0 + 4 * (int)threadIdx.x, m = n - i;
    if (m <= 0) return;
    const uint8_t *p = a + off * B + i;
    int s[4] = {0, 0, 0, 0};
#pragma unroll 8
    for (int b = 0; b < B; ++b) {
        const uint32_t w = load_bytes4(p + (int64_t)b * n, m);
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k] += (int)((w >> (8 * k)) & 0xffu);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (k < m) out[off + i + k] = (float)s[k] / (float)B;
}

// ---- launchers --------------------------------------------------------------
static int grid_for(int64_t n, int per_block, int cap) {
    const int64_t g = (n + per_block - 1) / per_block;
    return (int)std::max<int64_t>(1, std::min<int64_t>(g, cap));
}

hipError_t launch_features(const Plan &p, uint16_t *x, hipStream_t s) {
    const bool vec = (reinterpret_cast<uintptr_t>(x) & 15u) == 0;
    feature_kernel<<<p.n_tiles, kFeatThreads, 0, s>>>(p.d_rec, p.d_fd, p.d_tile, x, vec);
    return hipGetLastError();
}

hipError_t launch_mlp(const hp_mlp &net, const uint16_t *x, const float *y, int64_t rows, float *q, float *loss_sum,
                      bool backward, hipStream_t s) {
    if (backward) {
        // one workspace row per workgroup
        const int grid = grid_for((rows + kStepRows - 1) / kStepRows, 1, HP_MLP_PARTS);
        mlp_backward_kernel<<<grid, kBwdWaves * kWave, 0, s>>>(x, y, rows, net.params, net.w_bf16, net.partials);
        mlp_reduce_kernel<<<(HP_MLP_PARAMS + 1 + 63) / 64, 1024, 0, s>>>(net.partials, grid, net.grad, loss_sum);
    } else {
        mlp_forward_kernel<<<grid_for((rows + 31) / 32, kFwdWaves, 1024), kFwdWaves * kWave, 0, s>>>(
            x, rows, net.params, net.w_bf16, q);
    }
    return hipGetLastError();
}

hipError_t launch_adam(const hp_mlp &net, float lr, float beta1, float beta2, float eps, int64_t step, hipStream_t s) {
    const float c1 = 1.0f - powf(beta1, (float)step), c2 = 1.0f - powf(beta2, (float)step);
    adam_kernel<<<(HP_MLP_PARAMS + 255) / 256, 256, 0, s>>>(net.params, net.adam_m, net.adam_v, net.grad, lr, beta1,
                                                           beta2, eps, c1, c2, net.w_bf16);
    return hipGetLastError();
}

hipError_t launch_weights_to_bf16(const hp_mlp &net, hipStream_t s) {
    weights_to_bf16_kernel<<<(kOffB2 + 255) / 256, 256, 0, s>>>(net.params, net.w_bf16);
    return hipGetLastError();
}

hipError_t launch_init_chains(const Plan &p, const float *q, int chain_lo, int chain_hi, uint8_t *v, hipStream_t s) {
    if (chain_hi <= chain_lo) return hipSuccess;
    // chains per thread: as many as leave about eight workgroups per CU
    const int64_t want = (8 * (int64_t)p.cus + p.n_tiles - 1) / p.n_tiles;
    dim3 grid(p.n_tiles, (unsigned)std::max<int64_t>(1, std::min<int64_t>(chain_hi - chain_lo, want)));
    init_chains_kernel<<<grid, kTileGroups, 0, s>>>(q, p.d_fd, p.d_tile, p.B, chain_lo, chain_hi,
                                                    (uint32_t)(p.seed & 0xffffffffu), (uint32_t)(p.seed >> 32), v);
    return hipGetLastError();
}

hipError_t launch_chain_mean(const Plan &p, const uint8_t *a, float *out, hipStream_t s) {
    chain_mean_kernel<<<p.n_tiles, kTileGroups, 0, s>>>(a, p.d_fd, p.d_tile, p.B, out);
    return hipGetLastError();
}

}  // namespace hp
