// Sparsity-aware layer budgets (paper Alg. 1, SkewedCacheBudgetAllocation) in integer arithmetic.
// 1 - gamma'_l is proportional to n_l = sum_h nnz[l][h], so beta_l * m = n_l / N * alpha * L * m.
// The whole budget B_tot is apportioned by largest remainder and then clipped to
// [max(1, ceil(m/100)), m], the token form of the paper's clip(beta, 0.01, 1).
#include "common.h"
#include "internal.h"

namespace vlc {
namespace {

// Sum over the block: inside each wave with lane shifts, then over the four wave totals in LDS.
__device__ __forceinline__ uint64_t block_sum(uint64_t v, uint64_t* red) {
    for (int o = 32; o >= 1; o >>= 1) v += (uint64_t)__shfl_xor((unsigned long long)v, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = red[0] + red[1] + red[2] + red[3];
    __syncthreads();
    return v;
}

// One block per request.  A chain of a few loads and two block sums is all there is, so latency is what it costs: eight lanes
// share a layer's counts (all in flight together), then thread t owns layers t, t + 256, ...  (L <= kMaxLayers).
// Profiled, 32 layers of 32 heads 8.3 -> 5.4 us, 60 of 56 heads 11.4 -> 9.4 (a thread per layer, eight barriers per sum before).
// gamma, if asked for, is written from the counts as they come by: a launch of its own for it costs about 3 us.
__global__ __launch_bounds__(256) void allocate_kernel(const uint64_t* __restrict__ nnz, int L, int Hq, int m_max, int tau,
                                                       uint64_t alpha_num, uint64_t alpha_den,
                                                       const int32_t* __restrict__ lens, float* __restrict__ gamma, int32_t* __restrict__ k_out,
                                                       float* __restrict__ beta_out) {
    __shared__ uint64_t n_l[kMaxLayers];
    __shared__ uint64_t rem[kMaxLayers];
    __shared__ uint64_t quo[kMaxLayers];
    __shared__ uint64_t red[4];
    const int b = blockIdx.x;
    const int t = threadIdx.x;
    const ReqLen rl = request_len(lens, b, m_max, tau);
    const int m = rl.m;                                                     // this request's prompt length
    const uint64_t B_tot = alpha_num * (uint64_t)L * (uint64_t)m / alpha_den;   // floor(alpha L m) tokens for the request
    uint64_t local = 0;
    for (int l0 = 0; l0 < L; l0 += 32) {                    // block-uniform
        const int l = l0 + (t >> 3);
        uint64_t s = 0;
        if (l < L)
            for (int h = t & 7; h < Hq; h += 8) {
                const size_t x = ((size_t)b * L + l) * Hq + h;
                const uint64_t n = nnz[x];
                s += n;
                if (gamma) gamma[x] = gamma_of(n, rl);
            }
        for (int o = 4; o >= 1; o >>= 1) s += (uint64_t)__shfl_xor((unsigned long long)s, o, 64);
        if (l < L && (t & 7) == 0) { n_l[l] = s; local += s; }
    }
    const uint64_t N = block_sum(local, red);               // its barriers also publish n_l
    local = 0;
    for (int l = t; l < L; l += blockDim.x) {
        uint64_t q, r;
        if (N == 0) { q = B_tot / (uint64_t)L; r = 0; }
        else { const uint64_t prod = n_l[l] * B_tot; q = prod / N; r = prod % N; }
        quo[l] = q;
        rem[l] = r;
        local += q;
    }
    const uint64_t extra = B_tot - block_sum(local, red);   // < L tokens left after the floor quotas
    const int lo = max(1, (m + 99) / 100);
    for (int l0 = 0; l0 < L; l0 += 32) {                    // block-uniform: again eight lanes per layer
        const int l = min(l0 + (t >> 3), L - 1);
        // rank of layer l by (remainder descending, layer ascending)
        uint32_t rank = 0;
        const uint64_t r = rem[l];
        for (int x = t & 7; x < L; x += 8) rank += (rem[x] > r || (rem[x] == r && x < l)) ? 1u : 0u;
        for (int o = 4; o >= 1; o >>= 1) rank += (uint32_t)__shfl_xor((int)rank, o, 64);
        if (l0 + (t >> 3) >= L || (t & 7)) continue;
        uint64_t q = quo[l] + (rank < extra ? 1u : 0u);
        if (q < (uint64_t)lo) q = lo;
        if (q > (uint64_t)m) q = m;
        k_out[(size_t)b * L + l] = (int32_t)q;
        if (beta_out) beta_out[(size_t)b * L + l] = (float)((double)q / (double)m);
    }
}

}  // namespace

hipError_t launch_allocate(const vlc_shape& s, const uint64_t* nnz, int64_t alpha_num, int64_t alpha_den, float* gamma,
                           int32_t* k_out, float* beta_out, hipStream_t st) {
    allocate_kernel<<<s.B, 256, 0, st>>>(nnz, s.L, s.Hq, s.m, s.tau, (uint64_t)alpha_num, (uint64_t)alpha_den, s.lens, gamma,
                                         k_out, beta_out);
    return hipGetLastError();
}

}  // namespace vlc
