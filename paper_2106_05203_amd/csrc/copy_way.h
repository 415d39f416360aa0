// How ef21_set_state and ef21_get_state copy arrays (update.hip has the kernels).  Plain C++, so that the host can say for a shape which way it goes.
#pragma once
#include <cstdint>

namespace ef21 {

enum class CopyWay { kMemcpy, kCached, kStreamed };

// state: entries of the handle's own x, g_i and g; entries: of the arrays copied, `one` or several.  Several arrays go by one kernel, through the caches
// as long as the state and its copy fit the last one (256 MB, 64 million entries, and what a kernel finds there of the rest), past them beyond: what the
// cache kept of the copy would have to be written back while the next kernel reads.  One array alone goes by hipMemcpyAsync, whose launch is as good, where
// it is short or the state stays in the cache.  us, by hipMemcpyAsync, through the caches and past them: a step with supplied gradients and the copy of
// all three arrays out, n = 8, d = 2 million 82, 75 and 76; 2, 8 million 109, 101 and 108; 1, 13 million 142, 134 and 127; 8, 5 million 189, 179 and 165; 4, 12
// million 262, 263 and 226; all three in and a step, 2, 6 million 87, 85 and 98; 8, 4 million 155, 136 and 143; 8, 5 million 186, 178 and 171; 1, 40 million 417,
// 431 and 359; a step and the copy of x out, 4, 5 million 76, 76 and 79; 8, 7 million 157, 158 and 162; 20, 5 million 273, 274 and 278; 1, 18 million
// 117, 118 and 119; 1, 20 million 136, 136 and 130; 8, 11.2 million 249, 249 and 243; 4, 16 million 223, 224 and 214; 8, 20 million 473, 473 and 429; 1, 100
// million 714, 719 and 658.
constexpr int64_t kCopyStateStream = (int64_t)76 << 20, kCopyStream = (int64_t)10 << 20;
inline CopyWay copy_way(int64_t state, int64_t entries, bool one) {
    if (entries >= kCopyStream && state + entries >= kCopyStateStream) return CopyWay::kStreamed;
    return one ? CopyWay::kMemcpy : CopyWay::kCached;
}

// The mean of n rows of d entries, with a copy of them on the way or without.  A thread has one column (more threads, and up to 32 rows' loads in flight), or four
// where the rows and their copy do not stay in the last cache: there fewer, wider accesses past the caches are the better ones, loads from 38, stores from
// 67 million entries of x, g_i and g on (without a copy loads from 101).  set_state of x and g_i and a step, us, by hipMemcpyAsync and a mean, by one column and four a thread:
// n = 128, d = 65 537 79, 60 and 83; 128, 122 475 117, 76 and 130; 64, 180 001 76, 60 and 75; 128, 262 143 190, 140 and 175; 2, 6.1 million 89, 78 and
// 91; 20, 1.5 million 152, 120 and 124; 8, 4 million 165, 135 and 131; 8, 5 million 191, 171 and 157; 8, 7 million 268, 243 and 222; one worker of 20
// million 194, 188 and 229, of 30 million 287, 293 and 337.  The mean alone and a step, one column and four: 1, 122 475 25.1 and 24.6; 128, 122 475 71 and
// 96; 1, 9 million 91 and 84; 3, 4.2 million 76 and 74; 4, 12 million 188 and 189; 8, 4 million 115 and 117; 16, 1 million 70.4 and 71.0.
// Alone, past the caches in place of that: 8, 11.2 million 93 and 80, 2, 50 million 169 and 153, 4, 12 million 52 and 58.
enum class MeanWay { kMemcpy, kColumn, kQuad, kQuadStreamed };
constexpr int64_t kMeanQuad = (int64_t)36 << 20, kMeanStream = (int64_t)64 << 20, kMeanAlone = (int64_t)96 << 20, kMeanColumns = (int64_t)1 << 17;
inline MeanWay mean_way(int64_t n, int64_t d, bool copy) {
    const int64_t state = (n + 2) * d;
    if (!copy && state > kMeanAlone) return MeanWay::kQuadStreamed;
    if (!copy) return n >= 4 || d <= kMeanColumns ? MeanWay::kColumn : MeanWay::kQuad;
    if (n == 1 && state > kMeanStream) return MeanWay::kMemcpy;
    if (n <= 2 || state <= kMeanQuad) return MeanWay::kColumn;
    return state > kMeanStream ? MeanWay::kQuadStreamed : MeanWay::kQuad;
}

}  // namespace ef21
