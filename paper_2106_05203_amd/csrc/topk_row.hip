// Batched Top-k (Section 2.1 of the EF21 paper), one workgroup per row.
//
// The k largest magnitudes of a row are found by a radix select on the 31-bit magnitude key
// (fp32 bits with the sign cleared): three histogram passes (12 + 10 + 9 bits, LDS histograms)
// fix the key T of the k-th largest magnitude and the number q of entries equal to T that are
// still needed; an ordered emission then writes every entry with key > T and the first q
// entries with key == T, in ascending position order (ties go to the lower index).
// With `g_i != nullptr` the emission also updates the workers' state (TopkArgs::g_i).
#include "topk_row_impl.h"

namespace ef21 {
namespace {

// The row read from L2 in every pass: 16 KB of LDS, two workgroups per compute unit.
template <bool DIFF, int UPDATE>
__global__ __launch_bounds__(kRowThreads) void topk_row_kernel(TopkArgs p) {
    __shared__ RowShared s;
    row_topk<DIFF, UPDATE>(s, p, blockIdx.x);
}

template <int CACHE, bool DIFF, int UPDATE>
__global__ __launch_bounds__(kRowThreads) void topk_row_cached_kernel(TopkArgs p) {
    __shared__ RowShared s;
    __shared__ float cache[CACHE];
    row_topk_cached<DIFF, UPDATE>(s, cache, p, blockIdx.x);
}

template <int UPDATE>
__global__ __launch_bounds__(kRowThreads) void topk_row_parts_kernel(TopkArgs p) {
    __shared__ RowShared s;
    __shared__ float cache[kRowPartsMax];
    row_topk_parts<UPDATE>(s, cache, p, blockIdx.x);
}

template <int CACHE>
void launch_cached(const TopkArgs &p, hipStream_t stream) {
    const dim3 grid((unsigned)p.n), block(kRowThreads);
    const bool diff = p.b != nullptr, upd = p.g_i != nullptr;
    if (upd && diff) hipLaunchKernelGGL((topk_row_cached_kernel<CACHE, true, kAddUpdate>), grid, block, 0, stream, p);
    else if (upd) hipLaunchKernelGGL((topk_row_cached_kernel<CACHE, false, kClearUpdate>), grid, block, 0, stream, p);
    else if (diff) hipLaunchKernelGGL((topk_row_cached_kernel<CACHE, true, kNoUpdate>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((topk_row_cached_kernel<CACHE, false, kNoUpdate>), grid, block, 0, stream, p);
}

void launch_uncached(const TopkArgs &p, hipStream_t stream) {
    const dim3 grid((unsigned)p.n), block(kRowThreads);
    const bool diff = p.b != nullptr, upd = p.g_i != nullptr;
    if (upd && diff) hipLaunchKernelGGL((topk_row_kernel<true, kAddUpdate>), grid, block, 0, stream, p);
    else if (upd) hipLaunchKernelGGL((topk_row_kernel<false, kClearUpdate>), grid, block, 0, stream, p);
    else if (diff) hipLaunchKernelGGL((topk_row_kernel<true, kNoUpdate>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((topk_row_kernel<false, kNoUpdate>), grid, block, 0, stream, p);
}

}  // namespace

hipError_t launch_topk_row(const TopkArgs &p, hipStream_t stream) {
    const dim3 grid((unsigned)p.n), block(kRowThreads);
    const bool diff = p.b != nullptr, upd = p.g_i != nullptr;
    if (upd && p.g_i != (diff ? p.b : p.a)) return hipErrorInvalidValue;
    if (p.parts.part) {
        if (!diff || p.d > kRowPartsMax) return hipErrorInvalidValue;
        if (upd) hipLaunchKernelGGL((topk_row_parts_kernel<kAddUpdate>), grid, block, 0, stream, p);
        else hipLaunchKernelGGL((topk_row_parts_kernel<kNoUpdate>), grid, block, 0, stream, p);
        return hipGetLastError();
    }
    if (p.d <= kRowCacheShort) {
        launch_cached<kRowCacheShort>(p, stream);
    } else if (p.d <= kRowCache && p.n <= 256) {
        launch_cached<kRowCache>(p, stream);
    } else if (p.d <= kRowCache) {                    // more rows than compute units: see kRowCache
        launch_uncached(p, stream);
    } else {
        return hipErrorInvalidValue;                  // longer rows: launch_topk_row_reg, launch_topk_split
    }
    return hipGetLastError();
}

}  // namespace ef21
