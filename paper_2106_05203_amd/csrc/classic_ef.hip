// EF, the original error feedback (Algorithm 4 of the EF21 paper), kept beside EF21 as the method it is
// compared with.  One round at the current x, with the errors e_i in the place of EF21's g_i:
//   p_i = e_i + gamma grad f_i(x)   written over e_i (one fused multiply-add per entry; every entry changes,
//                                   unlike EF21's state, which changes in k places); on long rows, from the second
//                                   round on, by the Top-k's own pass over them (TopkArgs::add);
//   w_i = C(p_i)                    the library's Top-k on the rows of e;
//   e_i = p_i - w_i                 zero at the kept positions, written by the Top-k's emission;
//   x   = x - (1/n) sum_i w_i       the aggregation pass of Algorithm 2's line 8 from a zero vector, step 1.
#include "device_utils.h"
#include "kernels.h"

namespace ef21 {
namespace {

constexpr int kThreads = 256;

// All n * d entries in one stretch, four per thread and load; s may start at any 4-byte address (e is 16-byte aligned),
// the last one to three entries are taken one by one.
__global__ __launch_bounds__(kThreads) void ef_accumulate_kernel(const float *__restrict__ s, float *__restrict__ e,
                                                                 int64_t total, float gamma) {
    const int64_t stride = (int64_t)gridDim.x * kThreads, n4 = total / 4;
    const int64_t first = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    for (int64_t i = first; i < n4; i += stride) {
        const float4 sv = stream_load4_any(s + 4 * i);
        float4 ev = *reinterpret_cast<const float4 *>(e + 4 * i);
        ev.x = fmaf(gamma, sv.x, ev.x);
        ev.y = fmaf(gamma, sv.y, ev.y);
        ev.z = fmaf(gamma, sv.z, ev.z);
        ev.w = fmaf(gamma, sv.w, ev.w);
        *reinterpret_cast<float4 *>(e + 4 * i) = ev;
    }
    const int64_t left = 4 * n4 + first;
    if (left < total) e[left] = fmaf(gamma, s[left], e[left]);
}

unsigned blocks_for(int64_t items, int64_t cap) {
    int64_t b = (items + kThreads - 1) / kThreads;
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return (unsigned)b;
}

}  // namespace

hipError_t launch_ef_accumulate(const float *s, float *e, int32_t n, int64_t d, float gamma, hipStream_t stream) {
    const int64_t total = (int64_t)n * d;
    if ((uintptr_t)e % 16 != 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(ef_accumulate_kernel, dim3(blocks_for(total / 4, 8192)), dim3(kThreads), 0, stream, s, e, total, gamma);
    return hipGetLastError();
}

}  // namespace ef21
