// Batched Top-k (Section 2.1 of the EF21 paper) for rows of 512 to 61 440 entries and k <= 1024: one 1024-thread
// workgroup per row that keeps the whole row in its registers.
//
// The registers of a compute unit hold 512 KB, a row at most 240: every thread issues all of its loads (up to fifteen
// float4) at once and the row is never read or stored a second time.  A compute unit executes 64 lanes per clock, so
// every pass over a row of 50 000 entries costs a third of a microsecond per instruction and entry: after two short
// passes over the registers all work is done on a list of candidates in LDS.
//
// Against rows held in LDS as 16-bit prefixes of their keys, of which kept entries and the threshold's bin were read again
// (us a call, back to back): 100 x 50000, k = 500 19.8 -> 11.9; 20 x 20000, k = 200 15.0 -> 7.5; against full rows in LDS: 20 x 12000,
// k = 1000 14.9 -> 8.5; 600 x 16000, k = 80 46.2 -> 13.2; against many workgroups per row for differences (a step): 100 x 50000,
// k = 500 34.6 -> 26.0; 2 x 50000 23.2 -> 18.2.  What bounds it: 100 x 50000 takes 11 us in the kernel, of which the loads some 4, the two
// passes over the registers 1.5, and the rest a chain of fourteen barriers.
//
//   1  Every thread takes the largest magnitude key of each half of its registers: 2048 distinct entries (all entries of
//      rows of up to 4096).  The k-th
//      largest of them is no larger than the k-th largest entry of the row; a histogram over the 12 leading bits
//      (and, where the bin is crowded, the four bits behind them) gives `low`, the lower edge of its bin.
//   2  The quads that hold an entry of at least `low` (about one in twenty at k / d = 1 %) go to LDS with their
//      position: one atomic per wavefront, a bit mask per quad.
//   3  A histogram of the listed entries, (key - low) >> 14 (bins of 1/512 octave, a window of eight octaves), gives the
//      bin of the k-th largest magnitude; a crowded bin gets a histogram of its own.  The bin's entries (a handful) are
//      ranked against one another, larger key first, lower position first.
//   4  The kept entries set their bits in a bitmap of the row; a prefix sum over the bitmap gives each its place in
//      the ascending output.
// A list that overflows, a threshold beyond the window or more than 256 entries within four keys of it (rows with very many magnitudes
// alike, fewer than k non-zeros among them) leaves the threshold to a bisection of the keys over the registers.
#include "topk_row_impl.h"
#include "topk_row_reg_shared.h"

namespace ef21 {
namespace {

constexpr int kMaxQuads = 15;                   // per thread: 60 of 128 registers
static_assert((int64_t)kMaxQuads * kQuadStep == kRowRegMax, "the longest row fills the registers");
constexpr uint32_t kKeyEnd = 0x80000000u;       // beyond every key
constexpr int kWindowShift = 14, kFineShift = 2;
constexpr int kCrowded = 768;                   // maxima in a bin from which four more bits are worth two barriers
static_assert(kRegThreads == kRowThreads && kRegWaves == kRowWaves, "RegShared is the workgroup's");
static_assert(kRowRegMax <= 65536, "positions in 16 bits");

// Inclusive prefix sum over the wavefront, in vector instructions alone.
__device__ __forceinline__ uint32_t dpp_inclusive_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);     // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);     // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);     // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);     // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);    // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);    // row_bcast:31
    return v;
}

// Sum of `v` over the earlier threads of the workgroup.  One barrier; `waves` is free for the next use after another.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *waves) {
    const int lane = lane_id(), wave = wave_id();
    const uint32_t incl = dpp_inclusive_scan(v);
    if (lane == kWave - 1) waves[wave] = incl;
    __syncthreads();
    uint32_t w = dpp_inclusive_scan(waves[lane & (kRowWaves - 1)]);       // lanes 0..15: the wavefronts' running totals
    w = wave ? (uint32_t)__builtin_amdgcn_readlane((int)w, wave - 1) : 0u;
    return w + incl - v;
}

// Largest bin b of the histogram with count(bins > b) < need <= count(bins >= b): b, need - count(bins > b) and
// count(b) go to sh.bin, sh.need and sh.count (which stay as they are if need > total count).  The histogram is cleared.
// Two barriers.
template <int R>
__device__ __forceinline__ void select_and_clear(RegShared<R> &sh, uint32_t need) {
    static_assert(kBins == 4 * kRowThreads, "four bins per thread");
    const int tid = threadIdx.x;
    uint4 *mine = reinterpret_cast<uint4 *>(sh.hist) + (kRowThreads - 1 - tid);     // from the top
    const uint4 h = *mine;
    *mine = make_uint4(0u, 0u, 0u, 0u);
    const uint32_t total = h.x + h.y + h.z + h.w;
    const uint32_t above = block_exclusive_scan(total, sh.waves);
    if (above < need && need <= above + total) {            // exactly one thread
        const uint32_t c[4] = {h.w, h.z, h.y, h.x};
        uint32_t run = above, at = 0u, n = c[0];
#pragma unroll
        for (uint32_t j = 0; j < 3; ++j) {
            if (at == j && need > run + c[j]) {
                run += c[j];
                at = j + 1;
                n = c[j + 1];
            }
        }
        sh.bin = (uint32_t)(4 * (kRowThreads - 1 - tid) + 3) - at;
        sh.need = need - run;
        sh.count = n;
    }
    __syncthreads();
}

// hist[bin] += 1 for every lane with `has`: one atomic where all of them share a bin, as the lanes of rows with many
// magnitudes alike do, which would queue up at one address (4096 zeros: 7 us).
__device__ __forceinline__ void vote(uint32_t *hist, uint32_t bin, bool has) {
    const uint64_t all = __ballot(has);
    if (all == 0) return;
    const int first = __ffsll((long long)all) - 1;
    const uint32_t common = (uint32_t)__builtin_amdgcn_readlane((int)bin, first);
    if (__ballot(has && bin != common) == 0) {
        if (lane_id() == first) atomicAdd(&hist[common], popc64(all));
    } else if (has) {
        atomicAdd(&hist[bin], 1u);
    }
}

__device__ __forceinline__ uint32_t max_key(const float4 &v) {
    const uint32_t a = mag_key(v.x), b = mag_key(v.y), c = mag_key(v.z), e = mag_key(v.w);
    const uint32_t m = a > b ? a : b, n = c > e ? c : e;
    return m > n ? m : n;
}

// Exclusive prefix sum of the bitmap words' bit counts to sh.prefix.  Two barriers.
template <int R>
__device__ __forceinline__ void count_bitmap(RegShared<R> &sh) {
    constexpr int kMapWords = RegShared<R>::kMapWords;
    const int tid = threadIdx.x;
    const bool has = tid < kMapWords / 2;
    const uint32_t c0 = has ? (uint32_t)__popc(sh.bitmap[2 * tid]) : 0u;
    const uint32_t c1 = has ? (uint32_t)__popc(sh.bitmap[2 * tid + 1]) : 0u;
    const uint32_t run = block_exclusive_scan(c0 + c1, sh.waves);
    if (has) {
        sh.prefix[2 * tid] = run;
        sh.prefix[2 * tid + 1] = run + c0;
    }
    __syncthreads();
}

// The index of the row's message that launch_aggregate needs (TopkArgs::agg_start), after count_bitmap: a block of
// coordinates is a whole number of the bitmap's words.
template <int R>
__device__ __forceinline__ void write_index(const RegShared<R> &sh, const TopkArgs &p, int64_t row) {
    if (!p.agg_start) return;
    int32_t *start = p.agg_start + row * (p.agg_nblk + 1);
    for (int b = threadIdx.x; b <= (int)p.agg_nblk; b += kRowThreads)
        start[b] = b < (int)p.agg_nblk ? (int32_t)sh.prefix[b << (p.agg_shift - 5)] : (int32_t)p.k;
}

// `bits` without all but its `n` lowest set bits.
__device__ __forceinline__ uint32_t lowest_bits(uint32_t bits, uint32_t n) {
    uint32_t rest = bits;
    for (uint32_t i = 0; i < n && rest; ++i) rest &= rest - 1u;
    return bits ^ rest;
}

// The whole selection where the list did not serve: the key of the k-th largest magnitude by bisection, one count over the
// registers per step, then the bitmap from the registers and the output by its positions.  At least k entries reach `low`,
// `above` < k reach `end`; sh.bitmap is clear; all threads call.
template <int R, bool DIFF>
__device__ void select_by_bisection(RegShared<R> &sh, const TopkArgs &p, const float4 (&v)[R], uint32_t low, uint32_t end, uint32_t above,
                                    uint32_t max_of_thread) {
    const int tid = threadIdx.x, lane = lane_id();
    const uint32_t k = (uint32_t)p.k;
    constexpr int kMapWords = RegShared<R>::kMapWords;
    constexpr bool kHoldsRow = RegShared<R>::kHoldsRow;
    if constexpr (kHoldsRow) {
        __syncthreads();                                     // the list is done with
#pragma unroll
        for (int u = 0; u < R; ++u) *reinterpret_cast<float4 *>(sh.quads[u * kRowThreads + tid]) = v[u];
    }
    // The keys in the place of the values: those are read again at the end, from LDS or from memory.  (Opaque: kept from the passes before, the
    // compiler would hold keys beside values and spill.)
    uint32_t key[4 * R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const float w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            float f = w[t];
            asm volatile("" : "+v"(f));
            key[4 * u + t] = mag_key(f);
        }
    }
    __syncthreads();                                         // the counters are done with
    uint32_t *ties = sh.hist;
    for (int i = tid; i < kMapWords; i += kRowThreads) ties[i] = 0u;
    if (tid < 3) sh.probe[tid] = 0u;
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const uint32_t other = __shfl_xor(max_of_thread, o, kWave);
        max_of_thread = other > max_of_thread ? other : max_of_thread;
    }
    if (lane == 0) sh.waves[wave_id()] = max_of_thread;
    __syncthreads();
    for (int w = 0; w < kRowWaves; ++w) max_of_thread = sh.waves[w] > max_of_thread ? sh.waves[w] : max_of_thread;
    if (max_of_thread + 1u < end) {                          // no key beyond the largest
        end = max_of_thread + 1u;
        above = 0u;
    }
    __syncthreads();
    // the number of entries with a key of at least `from`; call number `i` of a sequence
    auto count = [&](uint32_t from, uint32_t i) {
        uint32_t c = 0u;
#pragma unroll
        for (int u = 0; u < 4 * R; ++u) c += popc64(__ballot(key[u] >= from));
        if (lane == 0 && c) atomicAdd(&sh.probe[i % 3u], c);
        __syncthreads();
        const uint32_t all = sh.probe[i % 3u];
        if (tid == 0) sh.probe[(i + 2u) % 3u] = 0u;           // read by all before this barrier, next used two calls on
        return all;
    };
    uint32_t T = low;                                        // T <= the threshold < end
    for (uint32_t i = 0; end - T > 1u; ++i) {
        const uint32_t mid = i == 0u ? T + 1u : T + (end - T) / 2u;      // zeros, and other rows whose ties lie at `low`
        const uint32_t c = count(mid, i);
        if (c >= k) {
            T = mid;
        } else {
            end = mid;
            above = c;
        }
    }
#pragma unroll
    for (int u = 0; u < R; ++u) {
        uint32_t gt = 0u, eq = 0u;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            gt |= key[4 * u + t] > T ? 1u << t : 0u;
            eq |= key[4 * u + t] == T ? 1u << t : 0u;
        }
        const uint32_t q = u * kRowThreads + tid, shift = 4u * (q & 7u);
        if (gt) atomicOr(&sh.bitmap[q >> 3], gt << shift);
        if (eq) atomicOr(&ties[q >> 3], eq << shift);
    }
    __syncthreads();
    {
        // the first k - above of the ties, by position
        const bool has = tid < kMapWords / 2;
        const uint32_t t0 = has ? ties[2 * tid] : 0u, t1 = has ? ties[2 * tid + 1] : 0u, n0 = (uint32_t)__popc(t0);
        const uint32_t before = block_exclusive_scan(n0 + (uint32_t)__popc(t1), sh.waves), quota = k - above;
        if (has) {
            sh.bitmap[2 * tid] |= lowest_bits(t0, quota > before ? quota - before : 0u);
            sh.bitmap[2 * tid + 1] |= lowest_bits(t1, quota > before + n0 ? quota - before - n0 : 0u);
        }
    }
    __syncthreads();
    count_bitmap(sh);
    write_index(sh, p, blockIdx.x);
    if ((uint32_t)tid < k) {                                 // one kept entry per thread
        int word = 0;                                        // the last word with prefix <= tid
        for (int step = 1024; step; step >>= 1)              // kMapWords <= 2048
            if (word + step < kMapWords && sh.prefix[word + step] <= (uint32_t)tid) word += step;
        const uint32_t bits = sh.bitmap[word], skip = (uint32_t)tid - sh.prefix[word];
        const uint32_t rest = bits ^ lowest_bits(bits, skip);
        const int64_t row = blockIdx.x, e = 32 * word + __ffs((int)rest) - 1, at = row * p.d + e;
        const float base = DIFF ? p.b[at] : 0.f;
        const float value = kHoldsRow ? (&sh.quads[0][0])[e] : DIFF ? p.a[at] - base : p.a[at];
        p.out_idx[row * p.k + tid] = (int32_t)e;
        p.out_val[row * p.k + tid] = value;
        if (p.g_i) p.g_i[at] = DIFF ? base + value : 0.f;
    }
}

// R quads per thread, d <= R * kQuadStep.
template <int R, bool DIFF>
__global__ __launch_bounds__(kRowThreads) void topk_row_reg_kernel(TopkArgs p) {
    __shared__ RegShared<R> sh;
    constexpr int kListMax = RegShared<R>::kListMax;
    const int64_t row = blockIdx.x;
    const int d = (int)p.d, tid = threadIdx.x, lane = lane_id();
    const uint32_t k = (uint32_t)p.k;
    const float *a = p.a + row * d;
    const float *b = DIFF ? p.b + row * d : nullptr;

    // ---- the row into registers; a quad beyond the end is read at the end and emptied below
    float4 v[R];
    auto at_of = [&](int u) {
        const int e = u * kQuadStep + tid * 4;
        return e < d - 4 ? e : d - 4;
    };
    if constexpr (!DIFF) {
#pragma unroll
        for (int u = 0; u < R; ++u) v[u] = stream_load4_any(a + at_of(u));
    } else {
        // of two arrays the registers hold one and a part: the subtrahend's quads in groups, one group ahead
        constexpr int G = 3, N = (R + G - 1) / G;
        float4 vb[2][G];
        auto issue = [&](int g) {
#pragma unroll
            for (int j = 0; j < G; ++j) {
                const int u = g * G + j;
                if (u < R) {
                    v[u] = stream_load4_any(a + at_of(u));
                    vb[g & 1][j] = load4_any(b + at_of(u));
                }
            }
        };
        issue(0);
#pragma unroll
        for (int g = 0; g < N; ++g) {
            if (g + 1 < N) issue(g + 1);
#pragma unroll
            for (int j = 0; j < G; ++j) {
                const int u = g * G + j;
                if (u < R) {
                    const float4 w = vb[g & 1][j];
                    v[u].x -= w.x;
                    v[u].y -= w.y;
                    v[u].z -= w.z;
                    v[u].w -= w.w;
                }
            }
        }
    }
    // cleared while the loads are in flight
    clear_shared(sh, tid);
    // Entries past the end become zeros at positions past the end: as the last of all ties they are never kept.
#pragma unroll
    for (int u = 0; u < R; ++u) {
        if (u * kQuadStep + (wave_id() + 1) * 4 * kWave > d) {
            const int over = u * kQuadStep + tid * 4 + 4 - d;              // entries of the quad past the end
            if (over > 0) {
                const float4 w = v[u];                                    // the row's last four
                v[u].x = over == 1 ? w.y : over == 2 ? w.z : over == 3 ? w.w : 0.f;
                v[u].y = over == 1 ? w.z : over == 2 ? w.w : 0.f;
                v[u].z = over == 1 ? w.w : 0.f;
                v[u].w = 0.f;
            }
        }
    }

    // ---- 1: a key that cannot lie above the k-th largest
    uint32_t max0 = 0u, max1 = 0u;
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const uint32_t m = max_key(v[u]);
        if (u < R / 2) max0 = m > max0 ? m : max0;
        else max1 = m > max1 ? m : max1;
    }
    __syncthreads();
    if constexpr (R == 1) {                                               // every entry: the bin of the k-th largest itself
        const uint32_t key[4] = {mag_key(v[0].x), mag_key(v[0].y), mag_key(v[0].z), mag_key(v[0].w)};
#pragma unroll
        for (int t = 0; t < 4; ++t) vote(sh.hist, key[t] >> 19, key[t] != 0u);
    } else {
        vote(sh.hist, max0 >> 19, max0 != 0u);
        vote(sh.hist, max1 >> 19, max1 != 0u);
    }
    __syncthreads();
    select_and_clear(sh, k);
    const uint32_t lead = sh.bin;
    uint32_t low = lead << 19;
    if (R > 1 && sh.count > (uint32_t)kCrowded) {
        const bool in0 = (max0 >> 19) == lead, in1 = (max1 >> 19) == lead;
        for (uint32_t i = 0; i < 16; ++i) {                               // counts from ballots: sixteen addresses
            const uint32_t c = popc64(__ballot(in0 && ((max0 >> 15) & 15u) == i)) +
                               popc64(__ballot(in1 && ((max1 >> 15) & 15u) == i));
            if (lane == 0 && c) atomicAdd(&sh.sub[i], c);
        }
        __syncthreads();
        uint32_t above = 0u;
        for (int i = 15; i >= 0; --i) {
            const uint32_t h = sh.sub[i];
            if (sh.need <= above + h) {
                low |= (uint32_t)i << 15;
                break;
            }
            above += h;
        }
    }

    const uint32_t max_of_thread = max0 > max1 ? max0 : max1;
    if (low == 0u) {                                                      // fewer than k non-zeros, or hardly more
        select_by_bisection<R, DIFF>(sh, p, v, 0u, kKeyEnd, 0u, max_of_thread);
        return;
    }

    // ---- 2: the quads that hold an entry of at least `low`
    {
        uint64_t has[R];
        uint32_t mine = 0u;
#pragma unroll
        for (int u = 0; u < R; ++u) {
            has[u] = __ballot(max_key(v[u]) >= low);
            mine += popc64(has[u]);
        }
        uint32_t at = 0u;
        if (lane == 0 && mine) at = atomicAdd(&sh.n_list, mine);
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const uint32_t i = at + lanes_below(has[u]);
            if (((has[u] >> lane) & 1u) && i < (uint32_t)kListMax) {
                *reinterpret_cast<float4 *>(sh.quads[i]) = v[u];
                sh.quad_at[i] = (uint16_t)(u * kRowThreads + tid);
            }
            at += popc64(has[u]);
        }
    }
    __syncthreads();
    const uint32_t n_list = sh.n_list;
    if (n_list > (uint32_t)kListMax) {
        select_by_bisection<R, DIFF>(sh, p, v, low, kKeyEnd, 0u, max_of_thread);
        return;
    }

    // ---- 3: the bin of the k-th largest, and its entries ranked.  Thread t takes the listed entries t, t + 1024, ...
    const float *flat = &sh.quads[0][0];
    const uint32_t n_flat = 4u * n_list;
    for (uint32_t i0 = 0; i0 < n_flat; i0 += kRowThreads) {
        const uint32_t i = i0 + tid, key = i < n_flat ? mag_key(flat[i]) : 0u;          // low > 0
        const uint32_t bin = (key - low) >> kWindowShift;
        vote(sh.hist, bin < (uint32_t)kBins - 1u ? bin : (uint32_t)kBins - 1u, key >= low);
    }
    __syncthreads();
    select_and_clear(sh, k);
    uint32_t need = sh.need, c = sh.count, width = kWindowShift;          // T's bin: keys [tie_lo, tie_lo + 2^width)
    uint32_t tie_lo = low + (sh.bin << kWindowShift);
    if (sh.bin == (uint32_t)kBins - 1u) {                                 // beyond the window
        select_by_bisection<R, DIFF>(sh, p, v, low, kKeyEnd, 0u, max_of_thread);
        return;
    }
    if (c > (uint32_t)kTieMax) {
        // Many entries just below what earlier iterations have sent, as EF21 leaves them: the bin's own histogram, four keys a bin
        // (100 x 50000, iterations of a sparse problem, us in this kernel: 22.2 and up to 44 with a bisection of the bin, 20.5 and up to
        // 27 so).
        static_assert(kWindowShift - kFineShift == 12 && kBins == 1 << 12, "the bin's keys fill the histogram");
        __syncthreads();                                                  // sh.bin, sh.need and sh.count have been read
        for (uint32_t i0 = 0; i0 < n_flat; i0 += kRowThreads) {
            const uint32_t i = i0 + tid, off = (i < n_flat ? mag_key(flat[i]) : 0u) - tie_lo;
            vote(sh.hist, off >> kFineShift, off < (1u << kWindowShift));
        }
        __syncthreads();
        select_and_clear(sh, need);
        need = sh.need;
        c = sh.count;
        width = kFineShift;
        tie_lo += sh.bin << kFineShift;
        if (c > (uint32_t)kTieMax) {
            select_by_bisection<R, DIFF>(sh, p, v, tie_lo, tie_lo + (1u << width), k - need, max_of_thread);
            return;
        }
    }
    for (uint32_t i = tid; i < n_flat; i += kRowThreads) {
        const uint32_t key = mag_key(flat[i]);
        if (key >= tie_lo) {
            const uint32_t e = 4u * sh.quad_at[i >> 2] + (i & 3u);
            if (key - tie_lo >= (1u << width)) {
                atomicOr(&sh.bitmap[e >> 5], 1u << (e & 31u));
            } else {
                const uint32_t at = atomicAdd(&sh.n_tie, 1u);
                sh.tie_key[at] = key;
                sh.tie_at[at] = e;
            }
        }
    }
    __syncthreads();
    {
        // c * c comparisons over all threads: thread t compares entry t mod c with one slice of the others
        const uint32_t parts = (uint32_t)kRowThreads / c, per = (c + parts - 1u) / parts;
        if ((uint32_t)tid < c * parts) {
            const uint32_t i = (uint32_t)tid % c, j0 = ((uint32_t)tid / c) * per;
            const uint32_t j1 = j0 + per < c ? j0 + per : c;
            const uint32_t key = sh.tie_key[i], e = sh.tie_at[i];
            uint32_t before = 0u;                            // entries that precede this one in the order
#pragma unroll 8
            for (uint32_t j = j0; j < j1; ++j) {
                const uint32_t kj = sh.tie_key[j], ej = sh.tie_at[j];
                before += (kj > key || (kj == key && ej < e)) ? 1u : 0u;
            }
            if (before) atomicAdd(&sh.tie_rank[i], before);
        }
    }
    __syncthreads();
    if ((uint32_t)tid < c && sh.tie_rank[tid] < need) {
        const uint32_t e = sh.tie_at[tid];
        atomicOr(&sh.bitmap[e >> 5], 1u << (e & 31u));
    }
    __syncthreads();

    // ---- 4: the places of the kept entries
    count_bitmap(sh);
    write_index(sh, p, row);
    int32_t *out_idx = p.out_idx + row * p.k;
    float *out_val = p.out_val + row * p.k;
    for (uint32_t i = tid; i < n_flat; i += kRowThreads) {
        const float value = flat[i];
        if (mag_key(value) >= low) {
            const uint32_t e = 4u * sh.quad_at[i >> 2] + (i & 3u), word = sh.bitmap[e >> 5], bit = 1u << (e & 31u);
            if (word & bit) {
                const uint32_t at = sh.prefix[e >> 5] + (uint32_t)__popc(word & (bit - 1u));
                out_idx[at] = (int32_t)e;
                out_val[at] = value;
                if (p.g_i) p.g_i[row * d + e] = DIFF ? b[e] + value : 0.f;      // Algorithm 2, line 6; Algorithm 4
            }
        }
    }
}

template <int R>
void launch(const TopkArgs &p, hipStream_t stream) {
    const dim3 grid((unsigned)p.n), block(kRowThreads);
    if (p.b) hipLaunchKernelGGL((topk_row_reg_kernel<R, true>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((topk_row_reg_kernel<R, false>), grid, block, 0, stream, p);
}

}  // namespace

hipError_t launch_topk_row_reg(const TopkArgs &p, hipStream_t stream) {
    if ((p.g_i && p.g_i != (p.b ? p.b : p.a)) || p.parts.part || p.d < kRowRegMin || p.d > kRowRegMax || p.k > kRowRegMaxK)
        return hipErrorInvalidValue;
    if (p.agg_start && (p.agg_shift < 5 || p.agg_nblk != ((p.d - 1) >> p.agg_shift) + 1)) return hipErrorInvalidValue;
    if (p.d <= kQuadStep) launch<1>(p, stream);
    else if (p.d <= 2 * kQuadStep) launch<2>(p, stream);
    else if (p.d <= 3 * kQuadStep) launch<3>(p, stream);
    else if (p.d <= 4 * kQuadStep) launch<4>(p, stream);
    else if (p.d <= 6 * kQuadStep) launch<6>(p, stream);
    else if (p.d <= 9 * kQuadStep) launch<9>(p, stream);
    else if (p.d <= 13 * kQuadStep) launch<13>(p, stream);
    else launch<15>(p, stream);
    return hipGetLastError();
}

}  // namespace ef21
