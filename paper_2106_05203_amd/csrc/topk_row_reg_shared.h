// The workgroup's LDS of the Top-k that holds a row in registers, and how it starts.  Plain C++ beside the kernel, so that
// the host can run every thread's part of it against the object's bounds: a store of zeros past an array is seen by no
// result on the GPU.
#pragma once
#include <cstdint>

#if defined(__HIPCC__)
#define EF21_BOTH_SIDES __host__ __device__ __forceinline__
#else
#define EF21_BOTH_SIDES inline
#endif

namespace ef21 {

constexpr int kRegThreads = 1024, kRegWaves = kRegThreads / 64;
constexpr int kQuadStep = kRegThreads * 4;      // entries between a thread's neighbouring quads
constexpr int kBins = 4096;
constexpr int kListMost = 4096;                 // listed quads
constexpr int kTieMax = 256;                    // entries of the threshold's bin that are ranked
constexpr int kSubBins = 16;
static_assert(kBins == 4 * kRegThreads, "four bins per thread");
static_assert(kTieMax <= kRegThreads && kSubBins <= kRegThreads, "an entry per thread, the other threads none");

// R quads per thread.  Rows of up to 16384 entries leave room for two workgroups per compute unit (1000 x 8193, k = 81:
// 25 us with one, 15 with two).
template <int R>
struct RegShared {
    static constexpr int kListMax = R <= 2 ? R * kRegThreads : R <= 4 ? 2560 : kListMost;
    static constexpr int kMapWords = R * kQuadStep / 32;
    static_assert(kMapWords % 2 == 0 && kMapWords <= 2 * kRegThreads, "two bitmap words per thread");
    static_assert(kMapWords <= kBins, "the bisection's map of ties lies over the histogram");
    static constexpr bool kHoldsRow = kListMax == R * kRegThreads;       // the list has room for every quad
    __attribute__((aligned(16))) uint32_t hist[kBins];
    __attribute__((aligned(16))) float quads[kListMax][4];
    uint32_t waves[kRegWaves];
    uint16_t quad_at[kListMax];                 // position / 4
    uint32_t tie_key[kTieMax], tie_at[kTieMax], tie_rank[kTieMax];
    uint32_t bitmap[kMapWords], prefix[kMapWords];
    uint32_t sub[kSubBins];
    uint32_t bin, need, count;                  // of the last selection
    uint32_t n_list, n_tie;
    uint32_t probe[3];
};

// Thread `tid`'s part of what has to be zero at the start: histograms, bitmap, ranks and counters.
template <int R>
EF21_BOTH_SIDES void clear_shared(RegShared<R> &sh, int tid) {
    for (int j = 0; j < 4; ++j) sh.hist[4 * tid + j] = 0u;
    for (int i = tid; i < RegShared<R>::kMapWords; i += kRegThreads) sh.bitmap[i] = 0u;
    if (tid < kTieMax) sh.tie_rank[tid] = 0u;
    if (tid < kSubBins) sh.sub[tid] = 0u;
    if (tid == 0) {
        sh.n_list = 0u;
        sh.n_tie = 0u;
        sh.bin = sh.count = 0u;                 // stand if fewer than k of the largest are no zeros
    }
}

}  // namespace ef21
