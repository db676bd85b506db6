// Sensitivity sampling (Algorithm 1, steps 3-5; proof of Theorem 2).
//
// p_i = s_i / S is realised exactly with integers: q_i = ceil(s_i 2^40)
// (exact, since s_i 2^40 is exact in float64 for a float32 s_i), C = inclusive
// prefix sum of q, Q = C[n-1].  Draw t uses the Philox4x32-10 block of
// counter (t, 0, 0) and key = seed, read as a 128-bit integer u, and picks
// the first index with C_i > floor(u Q / 2^128).  Weights are
// n_i Q / (m q_i), evaluated as two IEEE double products and one division
// (this file is built without floating-point contraction).
#include "gs_internal.hpp"

#include <algorithm>

namespace gs {

// Accepted sensitivities: [0, 1 + 2^-10].  A share is at most 1, but its
// float32 value can exceed 1 by a few ulps (a Gaussian alone on a ray scores
// (c rho) (1/A) with 1/A rounded); with n <= 2^24 - 2^16 values of at most
// 2^40 + 2^30 each, Q stays below 2^64.
constexpr float kSensMax = 1.0009765625f;   // 1 + 2^-10

// q_i = ceil(s_i 2^40) (0 for s_i = 0 and for values outside the accepted
// range, which k_quantize reports).
__device__ __forceinline__ uint64_t quantum(float x) {
    // (the integer value, below 2^42, read from the low bits of its sum with 2^52:
    // a conversion to 64 bits takes a dozen instructions)
    const double c = ceil((double)x * 0x1p40) + 0x1p52;
    return (x > 0.0f && x <= kSensMax) ? (uint64_t)__double_as_longlong(c) & ((1ull << 52) - 1ull) : 0ull;
}

// The inclusive prefix sum C of the quanta in blocks of kSampleBlock.  A
// sensitivity outside [0, 1 + 2^-10] (or NaN) could overflow Q: such a value
// gets q_i = 0 and marks its block's sum with kBadSum, which the host reads with
// Q and turns into an error (nothing is drawn then).  The quanta are formed
// twice instead of kept, which saves 16 bytes of traffic per Gaussian.
constexpr int kSampleThreads = 256, kSampleItems = 8, kSampleBlock = kSampleThreads * kSampleItems;
constexpr uint64_t kBadSum = 1ull << 63;    // (a block's sum stays below 2^52)

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
    for (int off = 32; off > 0; off >>= 1) v += (uint64_t)__shfl_xor((unsigned long long)v, off);
    return v;
}

// Block sums, and the outputs that start at zero.  (With fills, quanta and a
// general scan in launches of their own a draw of 100 000 from 10^6 took 127 us in
// nine launches, of which 68 us of kernels; five launches, 45 us: 74.)
__global__ __launch_bounds__(kSampleThreads) void k_sample_sums(const float *__restrict__ s, int64_t n,
                                                                uint64_t *__restrict__ sums,
                                                                uint32_t *__restrict__ counts,
                                                                int64_t *__restrict__ support) {
    __shared__ uint64_t wsum[kSampleThreads / 64];
    const int64_t lo = (int64_t)blockIdx.x * kSampleBlock;
    uint64_t sum = 0;
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kSampleItems; ++k) {
        const int64_t i = lo + k * kSampleThreads + threadIdx.x;
        if (i < n) {
            const float x = s[i];
            bad = bad || !(x >= 0.0f && x <= kSensMax);
            sum += quantum(x);
            counts[i] = 0u;
        }
    }
    sum = wave_sum_u64(sum);
    if (__any(bad)) sum |= kBadSum;
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t t = 0, flag = 0;
        for (int k = 0; k < kSampleThreads / 64; ++k) {
            t += wsum[k] & ~kBadSum;
            flag |= wsum[k] & kBadSum;
        }
        sums[blockIdx.x] = t | flag;
        if (blockIdx.x == 0) *support = 0;
    }
}

// Exclusive prefix sums of the block sums in place (one block);
// result = (Q, 1 if a block held a bad sensitivity).
__global__ __launch_bounds__(1024) void k_sample_prefix(uint64_t *__restrict__ sums, int nblk,
                                                        uint64_t *__restrict__ result) {
    __shared__ uint64_t wsum[16];
    const int per = (nblk + 1023) / 1024, lo = (int)threadIdx.x * per, hi = min(lo + per, nblk);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint64_t s = 0, flag = 0;
    for (int i = lo; i < hi; ++i) {
        s += sums[i] & ~kBadSum;
        flag |= sums[i] & kBadSum;
    }
    uint64_t incl = s;
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t x = (uint64_t)__shfl_up((unsigned long long)incl, off);
        if (lane >= off) incl += x;
    }
    if (lane == 63) wsum[w] = incl;
    const int bad = __syncthreads_or(flag != 0ull);
    uint64_t run = incl - s;
    for (int k = 0; k < w; ++k) run += wsum[k];
    for (int i = lo; i < hi; ++i) {
        const uint64_t c = sums[i] & ~kBadSum;
        sums[i] = run;
        run += c;
    }
    if (threadIdx.x == 1023) {
        result[0] = run;
        result[1] = bad ? 1ull : 0ull;
    }
}

__global__ __launch_bounds__(kSampleThreads) void k_sample_cdf(const float *__restrict__ s, int64_t n,
                                                               const uint64_t *__restrict__ sums,
                                                               uint64_t *__restrict__ C) {
    __shared__ uint64_t wsum[kSampleThreads / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t lo = (int64_t)blockIdx.x * kSampleBlock + (int64_t)threadIdx.x * kSampleItems;
    uint64_t q[kSampleItems], sum = 0;
#pragma unroll
    for (int k = 0; k < kSampleItems; ++k) {
        q[k] = lo + k < n ? quantum(s[lo + k]) : 0ull;
        sum += q[k];
    }
    uint64_t incl = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t x = (uint64_t)__shfl_up((unsigned long long)incl, off);
        if (lane >= off) incl += x;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    uint64_t run = sums[blockIdx.x] + incl - sum;
    for (int k = 0; k < w; ++k) run += wsum[k];
#pragma unroll
    for (int k = 0; k < kSampleItems; ++k) q[k] = run += q[k];
    if (lo + kSampleItems <= n) {
#pragma unroll
        for (int k = 0; k < kSampleItems; k += 2)
            *reinterpret_cast<ulonglong2 *>(C + lo + k) = make_ulonglong2(q[k], q[k + 1]);
    } else {
#pragma unroll
        for (int k = 0; k < kSampleItems; ++k)
            if (lo + k < n) C[lo + k] = q[k];
    }
}

int64_t sample_tmp_elems(int64_t n) { return (n + kSampleBlock - 1) / kSampleBlock; }

void launch_sample_cdf(const float *sens, int64_t n, uint64_t *C, uint64_t *sums, uint64_t *result, uint32_t *counts,
                       int64_t *support, hipStream_t st) {
    const unsigned nblk = (unsigned)sample_tmp_elems(n);
    hipLaunchKernelGGL(k_sample_sums, dim3(nblk), dim3(kSampleThreads), 0, st, sens, n, sums, counts, support);
    hipLaunchKernelGGL(k_sample_prefix, dim3(1), dim3(1024), 0, st, sums, (int)nblk, result);
    hipLaunchKernelGGL(k_sample_cdf, dim3(nblk), dim3(kSampleThreads), 0, st, sens, n, sums, C);
}

// Philox4x32-10 (Salmon et al., SC 2011): ten rounds of two 32x32->64
// multiplications with the round keys bumped by the golden-ratio and
// sqrt(3)-1 Weyl increments.
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c[1] ^ k0;
        const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c[3] ^ k1;
        c[1] = (uint32_t)p1;
        c[3] = (uint32_t)p0;
        c[0] = n0;
        c[2] = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// First index with C_i > target: the block from the block prefixes (in LDS, if
// they are at most kDrawSums) by halves, then four parts at a time, whose ends'
// loads do not wait for each other.  100 000 draws from 10^6 by halves alone, 20
// loads in a row: 15.3 us; so 13.7 (eight parts at a time, whose 28 loads per
// draw bind more than their waits: 17.5).
constexpr int kDrawSums = 2048;
__global__ __launch_bounds__(256) void k_draws(const uint64_t *__restrict__ C, const uint64_t *__restrict__ sums,
                                               const uint64_t *__restrict__ result, int64_t n, int64_t m,
                                               uint64_t seed, uint32_t *__restrict__ counts) {
    __shared__ uint64_t sh[kDrawSums];
    const int nblk = (int)((n + kSampleBlock - 1) / kSampleBlock);
    const bool in_lds = nblk <= kDrawSums;
    if (in_lds)
        for (int i = threadIdx.x; i < nblk; i += 256) sh[i] = sums[i];
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t Q = result[0];
    if (t >= m || Q == 0ull || result[1]) return;
    uint32_t c[4] = {(uint32_t)t, (uint32_t)((uint64_t)t >> 32), 0u, 0u};
    philox4x32_10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    const uint64_t u_lo = (uint64_t)c[0] | ((uint64_t)c[1] << 32);
    const uint64_t u_hi = (uint64_t)c[2] | ((uint64_t)c[3] << 32);
    // floor(u Q / 2^128) = hi word of (u_hi Q + floor(u_lo Q / 2^64))
    const uint64_t lo_hi = __umul64hi(u_lo, Q);
    const uint64_t hq_lo = u_hi * Q;
    const uint64_t hq_hi = __umul64hi(u_hi, Q);
    const uint64_t sum_lo = hq_lo + lo_hi;
    const uint64_t target = hq_hi + (sum_lo < hq_lo ? 1ull : 0ull);   // < Q
    // the last block that starts at or before the target: its end is past it
    int blo = 0, bhi = nblk - 1;
    while (blo < bhi) {
        const int mid = (blo + bhi + 1) >> 1;
        if ((in_lds ? sh[mid] : sums[mid]) <= target) blo = mid; else bhi = mid - 1;
    }
    // (C of the last Gaussian is Q: a part past the end counts as past the target)
    int64_t lo = (int64_t)blo * kSampleBlock;
    static_assert(kSampleBlock == 2048, "parts of 512, 128, 32, 8, 2 and 1");
#pragma unroll
    for (int part = 512; part >= 2; part /= 4) {
        int before = 0;
#pragma unroll
        for (int k = 1; k < 4; ++k) before += C[min(lo + k * part - 1, n - 1)] <= target ? 1 : 0;
        lo += before * part;
    }
    if (C[min(lo, n - 1)] <= target) ++lo;
    atomicAdd(&counts[lo], 1u);
}

void launch_draws(const uint64_t *C, const uint64_t *sums, const uint64_t *result, int64_t n, int64_t m,
                  uint64_t seed, uint32_t *counts, hipStream_t st) {
    hipLaunchKernelGGL(k_draws, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st, C, sums, result, n, m, seed,
                       counts);
}

// The support count is one atomic per block of a fixed grid: device-wide
// atomics on one address serialise (at n = 10^6 one per wave cost about 0.15 ms,
// one per 1024 Gaussians 10 us).
constexpr int kWeightBlocks = 256, kWeightThreads = 1024;

__global__ __launch_bounds__(kWeightThreads) void k_weights(const uint32_t *__restrict__ counts,
                                                            const float *__restrict__ sens,
                                                            const uint64_t *__restrict__ result, int64_t n, int64_t m,
                                                            double *__restrict__ w, int64_t *__restrict__ support) {
    __shared__ uint32_t wsup[kWeightThreads / 64];
    const double Q = (double)result[0];
    uint32_t sup = 0;
    for (int64_t i = (int64_t)blockIdx.x * kWeightThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kWeightThreads) {
        const uint32_t c = counts[i];
        double x = 0.0;
        if (c) {
            const double num = (double)c * Q;
            const double den = (double)m * (double)quantum(sens[i]);
            x = num / den;
            ++sup;
        }
        w[i] = x;
    }
    for (int off = 32; off > 0; off >>= 1) sup += (uint32_t)__shfl_xor((int)sup, off);
    if ((threadIdx.x & 63) == 0) wsup[threadIdx.x >> 6] = sup;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int k = 0; k < kWeightThreads / 64; ++k) t += wsup[k];
        if (t) atomicAdd((unsigned long long *)support, (unsigned long long)t);
    }
}

void launch_weights(const uint32_t *counts, const float *sens, const uint64_t *result, int64_t n, int64_t m,
                    double *weights, int64_t *support, hipStream_t st) {
    const int64_t blocks = std::min<int64_t>((n + kWeightThreads - 1) / kWeightThreads, kWeightBlocks);
    hipLaunchKernelGGL(k_weights, dim3((unsigned)blocks), dim3(kWeightThreads), 0, st, counts, sens, result, n, m,
                       weights, support);
}

}  // namespace gs
