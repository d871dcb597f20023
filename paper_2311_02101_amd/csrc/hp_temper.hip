// Replica exchange across the temperatures (the ensemble of free-energy
// targets).  Chain b of formula f samples the formula-RBM of temperature tau,
// whose visible marginal is p_tau(v) ~ exp(-F_tau(v)), F_tau the formula free
// energy (eq. 5): the sum over clauses of the clause free energy (eq. 1) of
// the clause's literal values (eq. 4).  A round pairs, in every formula, the
// k-th chain (by index) at tau with the k-th chain at tau + 1 for the pairs
// (tau, tau+1) of one parity and exchanges their temperatures with
// probability min(1, exp(D)),
//     D = F_tau(v_a) + F_tau+1(v_b) - F_tau(v_b) - F_tau+1(v_a),
// the draw U = (w >> 8) 2^-24 from word 0 of Philox4x32-10 at counter
// (t mod 2^32, a, 2^31 - 1, t div 2^32) with the sweep generator's key.
// In the size-clustered model every clause contributes the free energy of
// its own group's RBM.
#include <hip/hip_runtime.h>

#include "hp_internal.hpp"
#include "philox.hpp"

namespace hp {

constexpr int kFeThreads = 512;
constexpr uint32_t kSwapBlock = 0x7fffffffu;

__device__ __forceinline__ double softplus(double z) { return z > 0.0 ? z + log1p(exp(-z)) : log1p(exp(z)); }

// fe[tau][m] = -sum_l softplus(b_l + sum_k bit_k(m) W_kl) for patterns m < 2^K
__global__ void fe_table_kernel(const double *__restrict__ W, const double *__restrict__ b, int K, int L, int T,
                                double *__restrict__ fe) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= T * kPatterns) return;
    const int tau = i / kPatterns, m = i % kPatterns;
    double f = 0.0;
    if (m < (1 << K)) {
        const double *Wt = W + (size_t)tau * K * L;
        for (int l = 0; l < L; ++l) {
            double z = b[tau * L + l];
            for (int k = 0; k < K; ++k)
                if ((m >> k) & 1) z += Wt[k * L + l];
            f -= softplus(z);
        }
    }
    fe[i] = f;
}

// Size-clustered model: fe[tau][r] over the 248 pattern rows of the five
// groups (group K at row 2^K - 8), each with its own RBM.
__global__ void fe_table_clust_kernel(ClustRbm R, int T, double *__restrict__ fe) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= T * kClustThrRows) return;
    const int tau = i / kClustThrRows, row = i % kClustThrRows;
    const int K = 31 - __clz(row + 8), L = clust_hidden(K), m = row - ((1 << K) - 8);
    double f = 0.0;
    if (R.W[K - 3]) {
        const double *Wt = R.W[K - 3] + (size_t)tau * K * L;
        for (int l = 0; l < L; ++l) {
            double z = R.b[K - 3][tau * L + l];
            for (int k = 0; k < K; ++k)
                if ((m >> k) & 1) z += Wt[k * L + l];
            f -= softplus(z);
        }
    }
    fe[i] = f;
}

// The free energies that a round of one parity needs: of a chain at
// temperature tau only F_tau and that of its pair's other temperature, so two
// table columns instead of T.  out[item][part][0 / 1] = the sum over the
// part's clauses at the pair's lower / upper temperature; a chain whose
// temperature is in no pair of this parity writes nothing.
// A workgroup stages the chain's assignment and the two columns in LDS (a
// gather from global memory cost a cache line per literal); `parts`
// workgroups share a chain's clauses when there are few chains.
// kClust: a clause of length len reads row 2^K - 8 + m of the clustered
// table, K = max(len, 3), m its pattern padded to K inputs.
// Bound by the latency of a clause's dependent record, LDS gather and table
// reads: 32 chains of 12 288 clauses at 16 temperatures take 4.6 us, before
// 100 us with one workgroup of 256 threads per chain, gathers from global
// memory and all 16 columns.  Small formulas take fewer threads, at least one
// clause each (3000 formulas of 60 clauses x 8 chains, the whole round: 48 us with 256
// threads each, 74 with 512, 21 so).
template <bool kClust>
__global__ __launch_bounds__(kFeThreads) void free_energy_kernel(const FormulaDev *__restrict__ fd,
                                                                 const WorkItem *__restrict__ work,
                                                                 const uint4 *__restrict__ rec, int B, int T,
                                                                 int parity, uint32_t full,
                                                                 const int32_t *__restrict__ temp,
                                                                 const uint8_t *__restrict__ v,
                                                                 const double *__restrict__ fe,
                                                                 double *__restrict__ out) {
    constexpr int kRows = kClust ? kClustThrRows : kPatterns;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ double2 s_fe[kRows];
    __shared__ double2 s_part[kFeThreads / kWave];
    const WorkItem w = work[blockIdx.x];
    const int tau = temp[(int64_t)w.f * B + w.b];
    const int lo = tau - ((tau - parity) & 1);            // lower temperature of the pair
    if (lo < parity || lo + 1 >= T) return;
    const FormulaDev &f = fd[w.f];
    const int n = f.n, tid = threadIdx.x, NT = blockDim.x;
    const uint8_t *vb = v + f.var_off * B + (int64_t)w.b * n;
    for (int i = tid; i < kRows; i += NT)
        s_fe[i] = make_double2(fe[lo * kRows + i], fe[(lo + 1) * kRows + i]);
    for (int i = 4 * tid; i < n; i += 4 * NT) {
        uint32_t x = 0;
        if (i + 4 <= n) {
            __builtin_memcpy(&x, vb + i, 4);
        } else {
            for (int k = 0; i + k < n; ++k) x |= (uint32_t)vb[i + k] << (8 * k);
        }
        *reinterpret_cast<uint32_t *>(lds + i) = x & 0x01010101u;
    }
    __syncthreads();
    const uint4 *__restrict__ r = rec + f.clause_off;
    const int parts = (int)gridDim.y, part = (int)blockIdx.y;
    const int c_lo = (int)((int64_t)f.c * part / parts), c_hi = (int)((int64_t)f.c * (part + 1) / parts);
    double a0 = 0.0, a1 = 0.0;
#pragma unroll 2
    for (int c = c_lo + tid; c < c_hi; c += NT) {
        const uint4 q = r[c];
        const uint32_t len = rec_len(q.w), negm = rec_negm(q.w);
        const uint32_t e[7] = {q.x & 0xffffu, q.x >> 16, q.y & 0xffffu, q.y >> 16,
                               q.z & 0xffffu, q.z >> 16, q.w & 0xffffu};
        uint32_t m = 0;
#pragma unroll
        for (uint32_t k = 0; k < (uint32_t)kMaxK; ++k)
            if (k < len) m |= (uint32_t)lds[e[k] & 0x7fffu] << k;
        const uint32_t lenmask = (1u << len) - 1u;
        m = (m ^ negm) & lenmask;
        uint32_t row;
        if (kClust) {
            const uint32_t Kc = len < 3u ? 3u : len;
            m |= (m & 1u) ? (((1u << Kc) - 1u) & ~lenmask) : 0u;
            row = (1u << Kc) - 8u + m;
        } else {
            row = m | ((m & 1u) ? (full & ~lenmask) : 0u);   // padding copies of literal 0
        }
        const double2 x = s_fe[row];
        a0 += x.x;
        a1 += x.y;
    }
    for (int off = kWave / 2; off > 0; off >>= 1) {
        a0 += __shfl_xor(a0, off, kWave);
        a1 += __shfl_xor(a1, off, kWave);
    }
    if ((tid & (kWave - 1)) == 0) s_part[tid / kWave] = make_double2(a0, a1);
    __syncthreads();
    if (tid == 0) {
        double2 t = s_part[0];
        for (int i = 1; i < NT / kWave; ++i) {
            t.x += s_part[i].x;
            t.y += s_part[i].y;
        }
        *reinterpret_cast<double2 *>(out + 2 * ((size_t)blockIdx.x * parts + part)) = t;
    }
}

// One swap round per formula, one wave each: the wave lists the formula's
// chains by temperature (in chain order, ranks from lane masks), then lane p
// takes place p of the list; the k-th chain at the lower temperature of a
// pair meets the k-th at the upper one.  Latency bound (a chain of dependent
// loads, one Philox block and one exp per pair): 4.8 us for 32 chains at 16
// temperatures, before 46 us with one thread walking the pairs.
__global__ __launch_bounds__(kWave) void swap_kernel(int32_t *__restrict__ temp, const double *__restrict__ F, int B,
                                                     int T, int parts, int parity, const int64_t *__restrict__ t_ptr,
                                                     int32_t *__restrict__ list, uint32_t key0, uint32_t key1) {
    __shared__ int s_off[kMaxTemperTemps + 1];
    const int f = blockIdx.x, lane = threadIdx.x;
    int32_t *tn = temp + (size_t)f * B;
    int32_t *ls = list + (size_t)f * B;
    const uint64_t below = (1ull << lane) - 1ull;
    int off[kMaxTemperTemps + 1];                // first place of temperature k in the list
    for (int k = 0; k <= kMaxTemperTemps; ++k) off[k] = 0;
    for (int b0 = 0; b0 < B; b0 += kWave) {
        const int t = b0 + lane < B ? tn[b0 + lane] : -1;
#pragma unroll
        for (int k = 0; k < kMaxTemperTemps; ++k) off[k + 1] += __popcll(__ballot(t == k));
    }
#pragma unroll
    for (int k = 1; k <= kMaxTemperTemps; ++k) off[k] += off[k - 1];
    int at[kMaxTemperTemps];
#pragma unroll
    for (int k = 0; k < kMaxTemperTemps; ++k) at[k] = off[k];
    for (int b0 = 0; b0 < B; b0 += kWave) {
        const int t = b0 + lane < B ? tn[b0 + lane] : -1;
#pragma unroll
        for (int k = 0; k < kMaxTemperTemps; ++k) {
            const uint64_t m = __ballot(t == k);
            if (t == k) ls[at[k] + __popcll(m & below)] = b0 + lane;
            at[k] += __popcll(m);
        }
    }
    if (lane == 0)
        for (int k = 0; k <= kMaxTemperTemps; ++k) s_off[k] = off[k];
    __syncthreads();
    const uint64_t t = (uint64_t)*t_ptr;
    const double *Ff = F + 2 * (size_t)f * B * parts;
    const Key2 key{key0, key1 ^ (uint32_t)f};
    for (int p = lane; p < B; p += kWave) {
        int tau = 0;
        while (p >= s_off[tau + 1]) ++tau;
        const int k = p - s_off[tau];
        if (tau < parity || ((tau - parity) & 1) || tau + 1 >= T || k >= s_off[tau + 2] - s_off[tau + 1]) continue;
        const int a = ls[p], c = ls[s_off[tau + 1] + k];
        double a_lo = 0.0, a_hi = 0.0, c_lo = 0.0, c_hi = 0.0;
        for (int i = 0; i < parts; ++i) {
            const double *fa = Ff + 2 * ((size_t)a * parts + i), *fc = Ff + 2 * ((size_t)c * parts + i);
            a_lo += fa[0];
            a_hi += fa[1];
            c_lo += fc[0];
            c_hi += fc[1];
        }
        const double D = a_lo + c_hi - c_lo - a_hi;
        const uint4 rw = philox4x32_10_lane_key(make_uint4((uint32_t)t, (uint32_t)a, kSwapBlock,
                                                           (uint32_t)(t >> 32)), key);
        const double u = (double)(rw.x >> 8) * (1.0 / 16777216.0);
        if (u < exp(D < 0.0 ? D : 0.0)) {
            tn[a] = tau + 1;
            tn[c] = tau;
        }
    }
}

hipError_t launch_temper(Plan &p, const hp_state &st, int parity, hipStream_t s) {
    const size_t items = (size_t)p.F * p.B;
    const int rows = p.clust ? kClustThrRows : kPatterns;
    if (!p.d_fe) {
        hipError_t e = hipSuccess;
        if (!p.d_fe_chain) e = hipMalloc((void **)&p.d_fe_chain, items * kFeParts * 2 * sizeof(double));
        if (e == hipSuccess && !p.d_temp_list) e = hipMalloc((void **)&p.d_temp_list, items * sizeof(int32_t));
        if (e == hipSuccess) e = hipMalloc((void **)&p.d_fe, (size_t)p.T * rows * sizeof(double));
        if (e != hipSuccess) return e;
        if (p.clust)
            fe_table_clust_kernel<<<(p.T * rows + 255) / 256, 256, 0, s>>>(p.crbm, p.T, p.d_fe);
        else
            fe_table_kernel<<<(p.T * rows + 255) / 256, 256, 0, s>>>(p.d_W, p.d_b, p.K, p.L, p.T, p.d_fe);
    }
    // workgroups per chain: as many as give the device one wave of workgroups,
    // each with at least kFeThreads * 2 clauses of the largest formula
    int parts = 1;
    while (parts < kFeParts && items * parts * 2 <= (size_t)p.cus * 2 && p.max_c / (parts * 2) >= 2 * kFeThreads)
        parts *= 2;
    const dim3 grid((unsigned)items, (unsigned)parts);
    int threads = kFeThreads;
    while (threads > kWave && threads / 2 >= p.max_c) threads /= 2;
    const size_t lds = ((size_t)p.max_n + 15) / 16 * 16;
    if (p.clust)
        free_energy_kernel<true><<<grid, threads, lds, s>>>(p.d_fd, p.d_work_fb, p.d_rec, p.B, p.T, parity, 0u,
                                                               p.d_temp, st.v, p.d_fe, p.d_fe_chain);
    else
        free_energy_kernel<false><<<grid, threads, lds, s>>>(p.d_fd, p.d_work_fb, p.d_rec, p.B, p.T, parity,
                                                                (1u << p.K) - 1u, p.d_temp, st.v, p.d_fe,
                                                                p.d_fe_chain);
    swap_kernel<<<p.F, kWave, 0, s>>>(p.d_temp, p.d_fe_chain, p.B, p.T, parts, parity, st.t, p.d_temp_list,
                                      (uint32_t)(p.seed & 0xffffffffu), (uint32_t)(p.seed >> 32));
    return hipGetLastError();
}

}  // namespace hp
