// Exchange with the host heuristic (Sec. 3.4; the appendix program): count
// the current and the returned assignments of every chain, and keep, per
// formula, the B best of the 2B stacked rows (current first; a stable
// ascending sort of the counts, the last B rows kept, so equal counts favour
// the returned rows).  A kept row takes the variance average nu of the chain
// it came from ([nu; nu] stacked).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "hp_internal.hpp"

namespace hp {

// Assignments of both sets (0: current, 1: returned) as bits: word [set][g][i]
// holds variable i of chains 32 g .. 32 g + 31, so the count below judges a
// clause for 32 chains at once.  Also clears the counts.  A thread makes the
// words of four variables, one four-byte load per chain: bound by the latency of
// those loads (48 uneven formulas, 141 000 variables x 64 chains: 23 us, 18 MB
// read; 16 loads in flight instead of 8 changed nothing).
constexpr int kPackThreads = kTileVars / 4;

__global__ __launch_bounds__(kPackThreads) void pack_kernel(const FormulaDev *__restrict__ fd,
                                                            const VarTile *__restrict__ tile, int B, int64_t nv,
                                                            const uint8_t *__restrict__ v_cur,
                                                            const uint8_t *__restrict__ v_ret,
                                                            uint32_t *__restrict__ bits, int32_t *__restrict__ counts,
                                                            int64_t n_counts) {
    const int64_t blk = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    const int64_t blocks = (int64_t)gridDim.x * gridDim.y * gridDim.z;
    for (int64_t j = blk * kPackThreads + threadIdx.x; j < n_counts; j += blocks * kPackThreads) counts[j] = 0;
    const VarTile t = tile[blockIdx.x];
    const int n = fd[t.f].n;
    const int64_t off = fd[t.f].var_off;
    const int i = t.i0 + 4 * (int)threadIdx.x, m = min(4, n - i);
    if (m <= 0) return;
    const int g = (int)blockIdx.y, nb = min(32, B - 32 * g);
    const uint8_t *p = (blockIdx.z ? v_ret : v_cur) + off * B + (int64_t)g * 32 * n + i;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    auto add = [&](uint32_t x, int b) {
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] |= ((x >> (8 * k)) & 1u) << b;
    };
    if (m == 4) {
        // 16 loads in flight (rows past the last chain read the last one again)
#pragma unroll
        for (int b0 = 0; b0 < 32; b0 += 16) {
            if (b0 >= nb) break;
            uint32_t x[16];
#pragma unroll
            for (int b = 0; b < 16; ++b) __builtin_memcpy(&x[b], p + (int64_t)min(b0 + b, nb - 1) * n, 4);
#pragma unroll
            for (int b = 0; b < 16; ++b) add(x[b], b0 + b);
        }
    } else {
        for (int b = 0; b < nb; ++b) {
            uint32_t x = 0;
            for (int k = 0; k < m; ++k) x |= (uint32_t)p[(int64_t)b * n + k] << (8 * k);
            add(x, b);
        }
    }
    uint32_t *out = bits + ((int64_t)blockIdx.z * gridDim.y + g) * nv + off + i;
    for (int k = 0; k < m; ++k) out[k] = w[k];
}

// Satisfied clauses per chain of one set: a workgroup takes a tile of clauses
// for 32 chains.  The formula's words are staged in LDS (4 bytes per variable,
// 128 KB for the largest formula); a lane ORs its clause's literal words and
// adds the result, one bit per chain, into five bit-sliced counter planes (up
// to 31 clauses); the planes are then counted over the wave, one lane mask per
// plane and chain.  Bound by the LDS gathers and the counting of the
// planes: 31 us for both sets of the same batch (2 x 54 M clause tests), before
// 710 us with one chain per workgroup and a byte gather from global memory per
// literal.
// Fewer than 512 threads for small formulas, about eight clauses each (3000
// formulas of 60 clauses x 8 chains, the whole merge: 86 us with one chain per
// workgroup, 127 with 512 threads here and 16 slabs of columns below, 31 so).
constexpr int kCountThreads = 512;
constexpr int kPlanes = 5;
static_assert(kTileClauses / kCountThreads < (1 << kPlanes), "a lane's clauses fit its counter planes");

static int count_threads(int max_c) {
    int t = kWave;
    while (t < kCountThreads && t * 8 < max_c) t *= 2;
    return t;
}

__global__ __launch_bounds__(kCountThreads) void count_kernel(const FormulaDev *__restrict__ fd,
                                                              const ClauseTile *__restrict__ tile,
                                                              const uint4 *__restrict__ rec, int B, int64_t nv,
                                                              const uint32_t *__restrict__ bits, int64_t items,
                                                              int32_t *__restrict__ counts) {
    extern __shared__ __align__(16) uint32_t s_w[];
    __shared__ int32_t s_cnt[32];
    const ClauseTile t = tile[blockIdx.x];
    const FormulaDev &f = fd[t.f];
    const int tid = threadIdx.x, NT = blockDim.x, lane = tid & (kWave - 1), g = (int)blockIdx.y;
    const uint32_t *src = bits + ((int64_t)blockIdx.z * gridDim.y + g) * nv + f.var_off;
    for (int i = tid; i < f.n; i += NT) s_w[i] = src[i];
    if (tid < 32) s_cnt[tid] = 0;
    __syncthreads();
    const uint4 *__restrict__ r = rec + f.clause_off;
    const int c_hi = min(f.c, t.c0 + kTileClauses);
    uint32_t pl[kPlanes] = {};
#pragma unroll 2
    for (int c = t.c0 + tid; c < c_hi; c += NT) {
        const uint4 q = r[c];
        const uint32_t len = rec_len(q.w);
        const uint32_t e[7] = {q.x & 0xffffu, q.x >> 16, q.y & 0xffffu, q.y >> 16,
                               q.z & 0xffffu, q.z >> 16, q.w & 0xffffu};
        uint32_t sat = 0;
#pragma unroll
        for (uint32_t k = 0; k < (uint32_t)kMaxK; ++k)
            if (k < len) sat |= s_w[e[k] & 0x7fffu] ^ (0u - (e[k] >> 15));
#pragma unroll
        for (int j = 0; j < kPlanes; ++j) {
            const uint32_t carry = pl[j] & sat;
            pl[j] ^= sat;
            sat = carry;
        }
    }
    int32_t mine = 0;                            // lane b < 32: the wave's count of chain b
#pragma unroll
    for (int b = 0; b < 32; ++b) {
        int32_t n = 0;
#pragma unroll
        for (int j = 0; j < kPlanes; ++j) n += __popcll(__ballot((pl[j] >> b) & 1u)) << j;
        mine = lane == b ? n : mine;
    }
    if (lane < 32) atomicAdd(&s_cnt[lane], mine);
    __syncthreads();
    if (tid < 32 && 32 * g + tid < B)
        atomicAdd(&counts[blockIdx.z * items + (int64_t)t.f * B + 32 * g + tid], s_cnt[tid]);
}

// per formula: source row (0..2B-1) of each kept row
__global__ void select_kernel(const int32_t *__restrict__ cnt_cur, const int32_t *__restrict__ cnt_ret, int B,
                              int32_t *__restrict__ src) {
    constexpr int kStage = 1024;                 // counts staged in LDS (above it they are read from L2)
    __shared__ int32_t s_c[kStage];
    const int f = blockIdx.x;
    const int32_t *a = cnt_cur + (int64_t)f * B, *r = cnt_ret + (int64_t)f * B;
    const bool staged = 2 * B <= kStage;
    if (staged) {
        for (int j = threadIdx.x; j < 2 * B; j += blockDim.x) s_c[j] = j < B ? a[j] : r[j - B];
        __syncthreads();
    }
    for (int j = threadIdx.x; j < 2 * B; j += blockDim.x) {
        const int32_t cj = j < B ? a[j] : r[j - B];
        int rank = 0;
        if (staged) {
#pragma unroll 8
            for (int k = 0; k < 2 * B; ++k) rank += (s_c[k] < cj || (s_c[k] == cj && k < j)) ? 1 : 0;
        } else {
#pragma unroll 8
            for (int k = 0; k < B; ++k) rank += (a[k] < cj || (a[k] == cj && k < j)) ? 1 : 0;
#pragma unroll 8
            for (int k = 0; k < B; ++k) rank += (r[k] < cj || (r[k] == cj && k + B < j)) ? 1 : 0;
        }
        if (rank >= B) src[(int64_t)f * B + (rank - B)] = j;
    }
}

// Replaces the rows of v and nu by the kept ones, in place: a workgroup owns
// 64 columns of a formula, every wave reads its share of the kept rows there
// into registers, and after the barrier writes them, so nothing is staged in
// memory and each kept element is read and written once.  A row that keeps
// its place is left alone.  kPermRows rows per wave: up to kMergeRows chains.
// Bound by memory: 32 us for the same batch in FP32
// (up to 90 MB), before 125 us through staging buffers and two copies back.
// Above kMergeRows chains the staged form below remains.
constexpr int kPermWaves = 16, kPermRows = 16;
constexpr int kMergeRows = kPermWaves * kPermRows;

template <typename NuT>
__global__ __launch_bounds__(kPermWaves *kWave) void permute_rows_kernel(const FormulaDev *__restrict__ fd,
                                                                         const VarTile *__restrict__ tile, int B,
                                                                         const int32_t *__restrict__ src,
                                                                         uint8_t *v_cur, const uint8_t *v_ret,
                                                                         NuT *nu) {
    const VarTile t = tile[blockIdx.x];
    const int n = fd[t.f].n;
    const int64_t base = fd[t.f].var_off * B;
    const int i = t.i0 + (int)blockIdx.y * kWave + (int)(threadIdx.x & (kWave - 1));
    const bool on = i < n;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), waves = (int)blockDim.x / kWave;
    const int32_t *sf = src + (int64_t)t.f * B;
    uint8_t rv[kPermRows];
    NuT rn[kPermRows];
#pragma unroll
    for (int k = 0; k < kPermRows; ++k) {
        const int b = wave + k * waves;
        if (b < B) {
            const int j = sf[b];
            if (on && j != b) {
                rv[k] = j < B ? v_cur[base + (int64_t)j * n + i] : v_ret[base + (int64_t)(j - B) * n + i];
                rn[k] = nu[base + (int64_t)(j < B ? j : j - B) * n + i];
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPermRows; ++k) {
        const int b = wave + k * waves;
        if (b < B) {
            const int j = sf[b];
            if (on && j != b) {
                v_cur[base + (int64_t)b * n + i] = rv[k];
                if (j != b + B) nu[base + (int64_t)b * n + i] = rn[k];
            }
        }
    }
}

// gathers the kept rows (v and nu) into the staging buffers
__global__ void gather_rows_kernel(const FormulaDev *__restrict__ fd, const WorkItem *__restrict__ work, int B,
                                   const int32_t *__restrict__ src, const uint8_t *__restrict__ v_cur,
                                   const uint8_t *__restrict__ v_ret, const unsigned char *__restrict__ nu,
                                   int nu_bytes, uint8_t *__restrict__ v_out, unsigned char *__restrict__ nu_out) {
    const WorkItem w = work[blockIdx.x];           // destination row (formula w.f, chain w.b)
    const FormulaDev f = fd[w.f];
    const int j = src[(int64_t)w.f * B + w.b];
    const int64_t base = f.var_off * B;
    const uint8_t *vs = (j < B ? v_cur + base + (int64_t)j * f.n : v_ret + base + (int64_t)(j - B) * f.n);
    const int64_t nu_src = (base + (int64_t)(j % B) * f.n) * nu_bytes;
    const int64_t dst = base + (int64_t)w.b * f.n;
    for (int i = threadIdx.x; i < f.n; i += blockDim.x) v_out[dst + i] = vs[i];
    for (int64_t i = threadIdx.x; i < (int64_t)f.n * nu_bytes; i += blockDim.x)
        nu_out[dst * nu_bytes + i] = nu[nu_src + i];
}

// the words of a formula above 16384 variables take more than 64 KB of LDS
hipError_t set_merge_lds_limit() {
    return hipFuncSetAttribute((const void *)count_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                               kMaxVars * (int)sizeof(uint32_t));
}

hipError_t launch_merge(Plan &p, const hp_state &st, const uint8_t *cand, hipStream_t s) {
    const size_t items = (size_t)p.F * p.B;
    const size_t vbytes = (size_t)p.total_vars * p.B;
    const unsigned groups = (unsigned)((p.B + 31) / 32);
    // in place, a workgroup writes columns of v and nu that it alone reads: the
    // returned rows may be v itself, but not another part of the same memory
    const uintptr_t c = reinterpret_cast<uintptr_t>(cand);
    auto meets = [&](const void *q, size_t bytes) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(q);
        return c < a + bytes && a < c + vbytes;
    };
    const bool in_place =
        p.B <= kMergeRows && (cand == st.v || !meets(st.v, vbytes)) && !meets(st.nu, vbytes * st.nu_bytes);
    hipError_t e = hipSuccess;
    if (!p.d_mg_cnt) e = hipMalloc((void **)&p.d_mg_cnt, 3 * items * sizeof(int32_t));
    if (e == hipSuccess && !p.d_mg_bits)
        e = hipMalloc((void **)&p.d_mg_bits, 2 * (size_t)groups * p.total_vars * sizeof(uint32_t));
    if (e == hipSuccess && !in_place && !p.d_mg_v) e = hipMalloc((void **)&p.d_mg_v, vbytes);
    if (e == hipSuccess && !in_place && !p.d_mg_nu) e = hipMalloc((void **)&p.d_mg_nu, vbytes * 8);
    if (e != hipSuccess) return e;
    const size_t lds = (size_t)p.max_n * sizeof(uint32_t);
    int32_t *cnt_cur = p.d_mg_cnt, *cnt_ret = p.d_mg_cnt + items, *src = p.d_mg_cnt + 2 * items;
    pack_kernel<<<dim3(p.n_tiles, groups, 2), kPackThreads, 0, s>>>(p.d_fd, p.d_tile, p.B, p.total_vars, st.v, cand,
                                                                   p.d_mg_bits, p.d_mg_cnt, (int64_t)(2 * items));
    count_kernel<<<dim3(p.n_ctiles, groups, 2), count_threads(p.max_c), lds, s>>>(
        p.d_fd, p.d_ctile, p.d_rec, p.B, p.total_vars, p.d_mg_bits, (int64_t)items, p.d_mg_cnt);
    select_kernel<<<p.F, 256, 0, s>>>(cnt_cur, cnt_ret, p.B, src);
    if (in_place) {
        const int waves = std::min(kPermWaves, (p.B + kPermRows - 1) / kPermRows * 2);
        const dim3 grid(p.n_tiles, (std::min(p.max_n, kTileVars) + kWave - 1) / kWave);
        if (st.nu_bytes == 4)
            permute_rows_kernel<float><<<grid, waves * kWave, 0, s>>>(p.d_fd, p.d_tile, p.B, src, st.v, cand,
                                                                      reinterpret_cast<float *>(st.nu));
        else
            permute_rows_kernel<double><<<grid, waves * kWave, 0, s>>>(p.d_fd, p.d_tile, p.B, src, st.v, cand,
                                                                       reinterpret_cast<double *>(st.nu));
        return hipGetLastError();
    }
    gather_rows_kernel<<<(unsigned)items, 256, 0, s>>>(p.d_fd, p.d_work_fb, p.B, src, st.v, cand,
                                                        reinterpret_cast<const unsigned char *>(st.nu), st.nu_bytes,
                                                        p.d_mg_v, p.d_mg_nu);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(st.v, p.d_mg_v, vbytes, hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(st.nu, p.d_mg_nu, vbytes * st.nu_bytes, hipMemcpyDeviceToDevice, s);
    return e;
}

}  // namespace hp
