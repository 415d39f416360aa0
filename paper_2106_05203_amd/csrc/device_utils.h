// Wavefront-level helpers shared by the HIP kernels (gfx950: 64-wide wavefronts).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ef21 {

constexpr int kWave = 64;

// Magnitude key of Top-k: the fp32 bit pattern with the sign cleared.  For non-NaN values the
// unsigned order of keys is the order of |v|, +a and -a share a key, so do +0 and -0.
__device__ __forceinline__ uint32_t mag_key(float v) { return __float_as_uint(v) & 0x7fffffffu; }

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

// The wavefront's number in its workgroup, as a scalar: what is computed from it stays out of the vector registers.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)); }

// number of set bits of `mask` in lanes below the caller's
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ uint32_t popc64(uint64_t m) { return (uint32_t)__popcll(m); }

// Loads of streamed data (read once by the kernel, too large to stay in a cache): marked non-temporal
// so that the lines are not kept.  stream_load4 needs a 16-byte aligned address.
__device__ __forceinline__ float4 stream_load4(const float *p) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    const v4f t = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(p));
    return make_float4(t.x, t.y, t.z, t.w);
}
// The same for an address that is only 4-byte aligned (gfx950 loads 16 bytes from any dword address).
__device__ __forceinline__ float4 stream_load4_any(const float *p) {
    typedef float v4f __attribute__((ext_vector_type(4), aligned(4)));
    const v4f t = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(p));
    return make_float4(t.x, t.y, t.z, t.w);
}
// The same for data that is used again, and stores.
__device__ __forceinline__ float4 load4_any(const float *p) {
    typedef float v4f __attribute__((ext_vector_type(4), aligned(4)));
    const v4f t = *reinterpret_cast<const v4f *>(p);
    return make_float4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ void store4_any(float *p, const float4 &v) {
    typedef float v4f __attribute__((ext_vector_type(4), aligned(4)));
    v4f t;
    t.x = v.x;
    t.y = v.y;
    t.z = v.z;
    t.w = v.w;
    *reinterpret_cast<v4f *>(p) = t;
}
__device__ __forceinline__ void stream_store4_any(float *p, const float4 &v) {
    typedef float v4f __attribute__((ext_vector_type(4), aligned(4)));
    v4f t;
    t.x = v.x;
    t.y = v.y;
    t.z = v.z;
    t.w = v.w;
    __builtin_nontemporal_store(t, reinterpret_cast<v4f *>(p));
}
__device__ __forceinline__ float stream_load(const float *p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ int32_t stream_load(const int32_t *p) { return __builtin_nontemporal_load(p); }

// Derivative in z of the per-row loss of a linear model, z = a^T x:
//   kLossLogistic       log(1 + exp(-y z))  (Section 5, eq. (9)):   -y / (1 + exp(y z))
//   kLossLeastSquares   (z - y)^2           (Section 5.2):          2 (z - y)
//   kLossHalfSquare     z^2 / 2 (no target; its "gradient" is (1/m) A^T A x, used by the power iteration): z
__device__ __forceinline__ float loss_derivative(float y, float z, int loss) {
    if (loss == 2 /* kLossHalfSquare */) return z;
    return loss == 1 /* kLossLeastSquares */ ? 2.0f * (z - y) : -y / (1.0f + expf(y * z));
}

// Entry j of the power iteration's fixed start vector number `row`: positive, in [0.5, 1.5) from an integer hash of the
// position so that no two neighbours are alike, times scale = 1 / sqrt(d) (the vector's length is within [0.5, 1.5)).
__device__ __forceinline__ float power_start_entry(int64_t row, int64_t j, float scale) {
    uint32_t h = (uint32_t)j * 2654435761u + 0x9e3779b9u * (uint32_t)(row + 1);
    h ^= h >> 15;
    h *= 2246822519u;
    h ^= h >> 13;
    return (0.5f + (float)(h >> 8) * (1.0f / 16777216.0f)) * scale;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// Sum over each group of LANES consecutive lanes (16, 32 or 64), the same bits in every lane of the group, in
// vector instructions alone: neighbours by DPP inside a row of sixteen lanes, rows by the half-swaps of gfx950.
// (__shfl_xor goes through the LDS crossbar, six dependent round trips of it for a wavefront.)
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int LANES>
__device__ __forceinline__ float group_sum(float v) {
    static_assert(LANES == 16 || LANES == 32 || LANES == 64, "whole rows of sixteen lanes");
    v += dpp_move<0xB1>(v);                 // quad_perm [1,0,3,2]
    v += dpp_move<0x4E>(v);                 // quad_perm [2,3,0,1]
    v += dpp_move<0x141>(v);                // row_half_mirror: the other quad of eight lanes
    v += dpp_move<0x140>(v);                // row_mirror: the other eight lanes of the row
    if constexpr (LANES >= 32) {            // swaps the odd rows of one copy with the even rows of the other
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    if constexpr (LANES == 64) {            // swaps the upper half of one copy with the lower half of the other
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    return v;
}

// Place of the calling lane's item in a list whose length is `*counter` (LDS): the lanes of a wavefront that
// have an item (`has`) take consecutive places with ONE atomic for the wavefront.  Every lane of the wavefront
// must call; the result means something only where `has`.
__device__ __forceinline__ uint32_t wave_append(bool has, uint32_t *counter) {
    const uint64_t m = __ballot(has);
    if (m == 0) return 0u;
    const int first = __ffsll((long long)m) - 1;
    uint32_t base = 0u;
    if (lane_id() == first) base = atomicAdd(counter, popc64(m));
    return __shfl(base, first, kWave) + lanes_below(m);
}

// *p += v in LDS without the round trip of reading it first.  The LDS executes one wavefront's accesses in order, so where
// only that wavefront adds, and its lanes to different places at a time, the order of the additions is that of the code.
__device__ __forceinline__ void lds_add(float *p, float v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// All threads of the workgroup call.  Publishes what the workgroup has stored, draws a ticket of `counter`, and
// returns true in the workgroup that drew the last of `tickets` (it may then read what the others published).  flag: LDS.
// Every wavefront waits until its own stores and atomics have reached the L2 cache before the barrier: a barrier orders them, in the
// compiler's terms, by the caches that the workgroup shares, and is emitted without that wait.  One thread then fences for the
// workgroup: the device-scope fences write back and invalidate caches that the whole workgroup shares, so one of each is
// enough and sixteen wavefronts' worth would only queue up (one launch per iteration, us a step: n = 4, m = 250, d = 100 7.6 so, 10.8 with a
// fence by every wavefront; n = 20, m = 400, d = 300 19 and 84).
__device__ __forceinline__ bool draw_ticket(uint32_t *counter, uint32_t tickets, uint32_t *flag) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();                                     // release
        const uint32_t drawn = atomicAdd(counter, 1u);
        __threadfence();                                     // acquire
        *flag = drawn == tickets - 1u ? 1u : 0u;
    }
    __syncthreads();
    return *flag != 0u;
}

__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
    const int lane = lane_id();
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        uint32_t t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

}  // namespace ef21
