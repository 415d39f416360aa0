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

}  // namespace ef21
