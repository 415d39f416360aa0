// Last step of the dense gradient of eq. (9): one entry of grad f_i from the per-row-block partial sums
// of (sum_l r_l a_l).  Shared by the kernel that writes the gradient out and by the Top-k kernel that
// consumes it directly, so that both see the same bits.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace ef21 {

// The row blocks are added in fp64 in eight interleaved chains (block b into chain b mod 8, ascending), so that several
// threads can share a column; the chains in pairs.
__device__ __forceinline__ double dense_chains(const double (&s)[8]) {
    return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}

// sum / m + 2 lambda x_c / (1 + x_c^2)^2, rounded once to fp32.
__device__ __forceinline__ float dense_grad_of_sum(double sum, float x_c, int64_t m, float lambda) {
    const double xj = (double)x_c, q = 1.0 + xj * xj;
    return (float)(sum / (double)m + 2.0 * (double)lambda * xj / (q * q));
}

// part_w: the worker's partial sums [chunks][d]; c: the column.
__device__ __forceinline__ float dense_grad_entry(const float *__restrict__ part_w, int64_t chunks, int64_t d,
                                                  int64_t c, float x_c, int64_t m, float lambda) {
    double s[8] = {};
    int64_t b = 0;
    for (; b + 16 <= chunks; b += 16) {                 // sixteen loads in flight
        float p[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const float *block = part_w + (b + u) * d;  // the same for every lane
            p[u] = block[(uint32_t)c];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) s[u % 8] += (double)p[u];
    }
    auto rest = [&](auto count) {                       // up to `count` left; past the end: the last block, not added
        constexpr int kCount = decltype(count)::value;
        float p[kCount];
#pragma unroll
        for (int u = 0; u < kCount; ++u) {
            const float *block = part_w + (b + u < chunks ? b + u : chunks - 1) * d;
            p[u] = block[(uint32_t)c];
        }
#pragma unroll
        for (int u = 0; u < kCount; ++u)
            if (b + u < chunks) s[u % 8] += (double)p[u];
    };
    if (b + 4 < chunks) rest(std::integral_constant<int, 16>());
    else if (b + 1 < chunks) rest(std::integral_constant<int, 4>());
    else if (b < chunks) rest(std::integral_constant<int, 1>());
    return dense_grad_of_sum(dense_chains(s), x_c, m, lambda);
}

// The same for COLS columns from c0 on by THREADS / COLS threads per column (THREADS: the workgroup's), each with its share of
// the chains, AHEAD entries of each in flight; `lds`: 8 * COLS doubles.  Calls put(c, entry) for every column c < d by
// thread c - c0, and holds barriers.
template <int THREADS, int COLS, int AHEAD, class PutFn>
__device__ __forceinline__ void dense_grad_shared(const float *__restrict__ part_w, int64_t chunks, int64_t d, int64_t c0,
                                                  const float *__restrict__ x, int64_t m, float lambda, double *lds,
                                                  PutFn put) {
    constexpr int kShare = THREADS / COLS, kOwn = 8 / kShare, kAhead = AHEAD;
    static_assert(kShare * kOwn == 8, "every chain has one owner");
    static_assert(COLS % 64 == 0, "a wavefront's columns are one thread's share each");
    const int local = threadIdx.x % COLS, share = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / COLS));
    const int64_t c = c0 + local;
    const float x_c = share == 0 && c < d ? x[c] : 0.f;
    if (c < d) {
        double s[kOwn] = {};
        for (int64_t b = share * kOwn; b < chunks; b += 8 * kAhead) {
            float p[kAhead][kOwn];
#pragma unroll
            for (int a = 0; a < kAhead; ++a)
#pragma unroll
                for (int u = 0; u < kOwn; ++u) {
                    const int64_t at = b + 8 * a + u;                // past the end: the last block, as zero
                    const float *block = part_w + (at < chunks ? at : chunks - 1) * d;
                    p[a][u] = block[(uint32_t)c];
                }
#pragma unroll
            for (int a = 0; a < kAhead; ++a)
#pragma unroll
                for (int u = 0; u < kOwn; ++u) s[u] += b + 8 * a + u < chunks ? (double)p[a][u] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kOwn; ++u) lds[(share * kOwn + u) * COLS + local] = s[u];
    }
    __syncthreads();
    if (share == 0 && c < d) {
        double s[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) s[u] = lds[u * COLS + local];
        put((int)c, dense_grad_of_sum(dense_chains(s), x_c, m, lambda));
    }
    __syncthreads();
}

}  // namespace ef21
