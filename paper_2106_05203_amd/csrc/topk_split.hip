// Batched Top-k (Section 2.1 of the EF21 paper) for long rows: many workgroups per row, the row
// itself read ONCE.
//
// Same selection rule as the one-workgroup kernel (31-bit magnitude key, ties to the lower index,
// ascending output).  Three kernels:
//
//   collect   A key `key_lo` that (almost surely) at least k entries of the row reach is fixed first: from the
//             threshold key T of the previous call on the same quantity, lowered by a few per cent (warm start:
//             inside ef21_step consecutive iterations select nearly the same T), else from a fixed sample of the
//             row (64 evenly spaced pieces of 64 entries) that every workgroup of the row looks at.  Then each
//             wavefront streams a contiguous piece of the row and appends the entries with key >= key_lo
//             ("candidates", one or two per cent of the row) in position order to its own slot of the workspace,
//             counting them into the workgroup's LDS histogram of (key - key_lo) >> shift on the way (4096 bins;
//             keys beyond the window share the last bin).  The workgroup's histogram is added to the row's with
//             one atomic per non-empty bin.  No fences, no waiting.
//   count     Prologue of every workgroup: the bin that holds T, from the row's histogram.  Body, one wavefront
//             per slot: the slot's number of candidates in higher bins, and the candidates of T's bin (a handful)
//             appended to the row's short "tie list".
//   emit      Prologue: the tie list ranked in LDS (larger key first, lower position first) gives T and the number
//             q of entries equal to T to keep; the counts of the earlier slots give the output offset.  Body, one
//             wavefront per slot: ordered emission of the k kept entries (+ line 6 of Algorithm 2 on request).
//
// The guess can be wrong: fewer than k candidates, T beyond the histogram's window, or a crowded bin (more
// than kTieCap entries, i.e. very many equal magnitudes at the threshold).  After a warm start the count kernel's workgroups
// collect such a row again from the sample and then count it; a row that still fails is selected
// by the exact one-workgroup algorithm on the original data (one workgroup of the count or the emit kernel), so the
// result never depends on the guess.  Slots have the capacity of their piece, so any input fits.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "topk_row_impl.h"

namespace ef21 {
namespace {

constexpr int kBlk = kRowThreads;            // collect / rescue workgroups
constexpr int kBlkWaves = kBlk / kWave;
constexpr int kSample = 4096;                // sampled entries per row
constexpr int kSamplePer = kSample / kBlk;
constexpr int kSteps = 2;                    // steps of a collect group (loads in flight)
constexpr int kPieceLen = 64, kPieces = kSample / kPieceLen;   // a wavefront's load is one piece
constexpr int kMaxSlots = 4096;              // slots (wavefront pieces) per row
constexpr int kCandThreads = 1024;           // count / emit workgroups: one wavefront per slot
constexpr int kCandWaves = kCandThreads / kWave;
constexpr int kBins1 = 1 << kBits1;
constexpr int kHistBins = 4096;              // bins of the candidates' histogram
static_assert(kHistBins == kBins1, "the candidates' histogram lives in RowShared::hist");
static_assert(kCandThreads == kRowThreads && kBlk == kRowThreads, "the rescue runs the one-workgroup algorithm");
// Bin width of the candidates' histogram as a shift of the key.  From a sample T lies up to a fraction of an octave
// above key_lo: the window is one octave (2^23 keys).  After a warm start key_lo is kWarmBelow keys (1/8 octave,
// 8.3 %) below the previous T and the window half an octave, so a threshold between 0.92 and 1.3 times the
// previous one is found by the first pass: narrower bins, fewer entries to rank.  A candidate costs little (an
// 8-byte store), a failed guess a second pass over the row, hence the generous margin; where T has just moved both are wider, see
// warm_start.
// That is where many entries are kept.  Where few are, T of a heavy-tailed row lies up to an octave above the sample's
// bound, and a row that failed so once starts from a sample, and can fail again, in every later call (n = 15, d = 5
// million, k = 5000, Student-t gradients: 13 ms an iteration against 0.14, all of it the exact algorithm on one row), so
// the window may be wider there: widest_cold and widest_warm.  It is so only where T's bin then holds no more than
// kBinEntries entries, by the sample's density around T or, after a warm start, by what T's bin held in the call before:
// heavy and Gaussian tails always, but the largest of 3 million uniform entries share a few bins, and a bin of more than
// kTieCap different keys costs the exact algorithm (n = 1, d = 3 million, k = 1000, U(0, 1): 5.4 ms in the widest window,
// 37 us in one of an octave).  The limit leaves a factor of 16 for a density that is uneven inside 1/16 octave.
constexpr uint32_t kBinEntries = 64;
__host__ __device__ inline uint32_t widest_cold(int64_t k, int64_t d) {
    if (k <= 4096) return 13u;                                    // four octaves
    if (k <= 131072 && k * 200 < d) return 12u;                   // two
    return k <= 400000 ? 11u : 10u;                               // one; half, where a wider bin would be crowded
}
__host__ __device__ inline uint32_t widest_warm(int64_t k, int64_t d) {
    if (k > 1500000) return 9u;
    const uint32_t s = widest_cold(k, d);
    return s > 10u ? s - 1u : 10u;
}
// in_bin: entries of T's bin, 2^used keys wide, in this call (at most kTieCap, or kCrowdedBin)
constexpr uint32_t kCrowdedBin = 1u << 16;
__device__ __forceinline__ uint32_t warm_shift(int64_t k, int64_t d, uint32_t in_bin, uint32_t used) {
    uint32_t s = widest_warm(k, d);
    while (s > 10u && (in_bin << s) >> used > kBinEntries) --s;
    return s;
}
constexpr uint32_t kWarmBelow = 1u << 20;
// A threshold that has just moved by more than three quarters of that, or that is the first one, may well move again by more than it
// allows.  The steps of EF21 from a fresh state on gradients that stay alike keep k entries more each: at k = 5 per
// cent of a Gaussian row T falls by 16 per cent, then 12, 11, 10 ..; the errors of EF grow from zero by 100 per cent, 50, 33 ..; and a
// failed guess costs twice the call.  After a fall, half an octave of margin brings two to seven times the candidates
// instead; after either, a window of two octaves (bins of 2^12 keys) or one, unless T's bin would be crowded, costs next to nothing.  The first
// ten steps, us each, before and now: EF21 on n = 8, d = 10^6, k = 10^4 52 and 47; n = 5, d = 10^6, k = 50 000 67 and 51; n = 8, d = 11.2 million,
// k = 112 000 347 and 279.
// Not where the bin was crowded, with equal magnitudes then (crowded): a wider one can take in different ones beside them, and that row goes to the
// exact algorithm (2 million of 3 million equal, 100 000 others 2560 keys away: 9.5 ms a step, 0.11 without).
// (From half of the margin on, thresholds that fall by ever less got the wide one for nothing: n = 20, d = 5 million, k = 50 000, the sixth and the eighth step from a
// fresh state on two gradients in turn 312 us each, 258 so.)
constexpr uint32_t kMoved = 3u << 18, kWarmBelowWide = 1u << 22, kWideEntries = 256u;
constexpr uint32_t kWideStart = 0x100u;      // flag in RowInfo::warm_s: the wide margin, which takes a window of an octave
__device__ __forceinline__ uint32_t warm_start(int64_t k, int64_t d, bool crowded, uint32_t in_bin, uint32_t used, bool before, uint32_t T_before, uint32_t T,
                                               bool errors) {
    uint32_t s = warm_shift(k, d, crowded ? kBinEntries : in_bin, used);              // crowded: no wider (narrower would not help)
    const bool fell = !before || T + kMoved < T_before, rose = !before || T > T_before + kMoved;
    if (!crowded && (fell || rose)) {
        // (EF21's falling threshold comes to where the entries are closer together: two octaves took a third more time in a run that had kept
        // all entries; the errors of EF fall when a run starts again, and grow then)
        for (uint32_t wide = before && fell && !errors ? 11u : 12u; wide > s && wide > 10u; --wide)
            if ((in_bin << wide) >> used <= kWideEntries) s = wide;
    }
    return fell && s >= 11u ? s | kWideStart : s;
}
// lower bound of the candidates' keys and bin width of a start from threshold T, noted as `start`
__device__ __forceinline__ void start_from(uint32_t T, uint32_t start, uint32_t *key_lo, uint32_t *shift) {
    const uint32_t below = start & kWideStart ? kWarmBelowWide : kWarmBelow;
    *key_lo = T > below ? T - below : 0u;
    *shift = start & ~kWideStart;
}
constexpr int kTieCap = 1024;                // entries of T's bin that are ranked directly (one per thread)
constexpr int kWarmSlots = 1;                // remembered thresholds per row (TopkArgs::warm = 1 .. kWarmSlots)
enum CollectMode { kColdPass = 0, kWarmPass = 1, kSecondPass = 2 };
// TopkArgs::add, and how the sums are stored: as lines that stay in the caches for the next round, or past them.
enum AddMode { kNoAdd = 0, kAddKept = 1, kAddStreamed = 2 };

struct __attribute__((aligned(64))) RowInfo {     // one cache line per row
    uint32_t key_lo, shift;       // lower bound of the candidate keys and bin width
    uint32_t key_lo2, shift2;     // ... of the row collected again, valid if use2
    uint32_t use2;                // the count kernel collected this row again: its histogram is hist_b
    uint32_t warm_used;           // the first pass started from a remembered threshold
    uint32_t failed;              // kRowFailed: the row went to the exact one-workgroup algorithm in the count kernel;
                                  // kRowCrowded: T's bin holds more than kTieCap candidates (see tie_min, tie_max);
                                  // kRowPending: not known yet
    uint32_t bin_a, need_a;       // bin of T; entries still needed from that bin
    uint32_t ntie;                // length of the tie list
    uint32_t arrived;             // workgroups of the count kernel that have collected the row again, then also the slot
                                  // blocks that have been taken to be counted
    uint32_t warm_T[kWarmSlots];  // threshold T of the last call (also with warm == 0)
    uint32_t warm_s[kWarmSlots];  // bin width for the next warm start from it, with kWideStart; 0: there is none to start from
    uint32_t tie_min, tie_max;    // crowded bin: smallest and largest key in it.  Equal: T is that key (many equal
                                  // magnitudes at the threshold, e.g. zeros), no ranking needed.  Different: the
                                  // exact one-workgroup algorithm, in the emit kernel.
};
enum { kRowFine = 0, kRowFailed = 1, kRowCrowded = 2, kRowPending = 3 };
static_assert(sizeof(RowInfo) == 64, "one cache line");

// How a sample is read, from k and d alone (set on the host: double precision in every wavefront cost half a microsecond).
struct SampleRule {
    uint32_t r;          // the r-th largest sampled key is, except with negligible probability, not above the k-th largest
                         // key of the row; above kSample: no bound
    uint32_t mid;        // where T is expected among the sampled keys
    uint32_t widest;     // widest_cold
    uint32_t most, most_next;   // samples in T's 2^19 keys up to which the bins are that wide, and half as wide
};
SampleRule sample_rule(int64_t k, int64_t d) {
    SampleRule q{};
    const double ns = (double)std::min<int64_t>(d, kSample), mu = (double)k * ns / (double)d;
    // mean + 5 standard deviations + 8 of the number of sampled entries among the row's top k (a binomial with mean mu)
    q.r = d <= kSample ? (uint32_t)k : (uint32_t)std::ceil(mu + 5.0 * std::sqrt(mu) + 8.0);
    q.mid = std::max<uint32_t>(1u, std::min<uint32_t>(q.r, (uint32_t)(mu + 0.5)));
    q.widest = widest_cold(k, d);
    // a sample in 2^19 keys stands for d / ns / 2^19 entries per key; never narrower than 2^11 keys
    auto most = [&](uint32_t s) { return (uint32_t)(s <= 11u ? (double)kSample : (double)kBinEntries * 524288.0 / (double)(1u << s) * ns / (double)d); };
    q.most = most(q.widest);
    q.most_next = most(q.widest - 1u);
    return q;
}

struct Ws {
    uint32_t *hist_a, *hist_b;            // [n][kHistBins] each, kept zero between calls
    RowInfo *info;                        // [n]
    uint32_t *slot_cnt, *slot_above;      // [n][nslot] candidates of a slot; those in bins above T's
    uint32_t *slot_inbin;                 // [n][nslot] those in T's bin (written for crowded bins only)
    uint2 *tie;                           // [n][kTieCap] (position, key) of the candidates in T's bin
    uint2 *cand;                          // [n][nslot][L] (position, value bits) of the candidates
    // Algorithm 3 only (launch_topk_split_pair), the caller's:
    float *resid;                         // [n][nslot][L] what the rounding of a difference took away (nullptr: not kept)
    double *kept;                         // [n][nslot] sum of the squares of the kept entries, unrounded
    int64_t L;                            // entries per wavefront piece = slot capacity
    int64_t nslot;                        // pieces per row
    int64_t G;                            // collect workgroups per row
    SampleRule rule;                      // of the call's k and d
};

size_t align256(size_t b) { return (b + 255) / 256 * 256; }

void plan(int32_t n, int64_t d, Ws *w) {
    // One 1024-thread workgroup per compute unit.  (Two, one step of loads ahead each or two, us a step: n = 15, d = 5
    // million, k = 5000 147 and 145 against 136; n = 8, d = 11.2 million, k = 112000 225 and 222 against 212; ef21_topk of 10 rows
    // of 7 million 69 and 72 against 64; shorter inputs lose more, each workgroup repeats the sampling prologue.)
    int64_t max_g = 256 / n;
    if (max_g < 1) max_g = 1;
    if (max_g > kMaxSlots / kBlkWaves) max_g = kMaxSlots / kBlkWaves;
    // At least 2048 entries per piece; 1024 where that would leave most compute units idle (up to 2 million entries: n = 10,
    // d = 10^5, k = 5000 21.6 us a call against 20.1; at 3 to 5 million 0.5 us are lost to the longer merge; many
    // short rows have a workgroup each anyway).
    const int64_t piece = n <= 64 && (int64_t)n * d <= 2000000 ? 1024 : 2048;
    int64_t g = (d + kBlkWaves * piece - 1) / (kBlkWaves * piece);
    if (g > max_g) g = max_g;
    if (g < 1) g = 1;
    const int64_t pieces = g * kBlkWaves;
    int64_t L = (d + pieces - 1) / pieces;
    const int64_t unit = piece == 2048 ? 2048 : 512;
    L = (L + unit - 1) / unit * unit;        // whole load groups (2 steps of 64 lanes x 4 entries), and whole
                                             // blocks of the aggregation's message index (256 or 512 coordinates)
    w->L = L;
    w->nslot = (d + L - 1) / L;
    w->G = (w->nslot + kBlkWaves - 1) / kBlkWaves;
}

size_t layout(int32_t n, int64_t d, char *base, Ws *w) {
    Ws tmp;
    plan(n, d, &tmp);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *p = base ? base + off : nullptr;
        off += align256(bytes);
        return p;
    };
    // the leading part (histograms, row records) starts at zero: launch_topk_split_reset
    char *ha = take(sizeof(uint32_t) * (size_t)n * kHistBins);
    char *hb = take(sizeof(uint32_t) * (size_t)n * kHistBins);
    char *inf = take(sizeof(RowInfo) * (size_t)n);
    const size_t slots = sizeof(uint32_t) * (size_t)n * tmp.nslot;
    char *s0 = take(slots), *s1 = take(slots), *s2 = take(slots);
    char *tl = take(sizeof(uint2) * (size_t)n * kTieCap);
    char *cd = take(sizeof(uint2) * (size_t)n * tmp.nslot * tmp.L);
    if (w) {
        *w = tmp;
        w->hist_a = (uint32_t *)ha; w->hist_b = (uint32_t *)hb;
        w->info = (RowInfo *)inf;
        w->slot_cnt = (uint32_t *)s0; w->slot_above = (uint32_t *)s1; w->slot_inbin = (uint32_t *)s2;
        w->tie = (uint2 *)tl;
        w->cand = (uint2 *)cd;
        w->resid = nullptr;
        w->kept = nullptr;
        w->rule = SampleRule{};
    }
    return off;
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// Bin of a candidate key (key >= key_lo) in the candidates' histogram.
__device__ __forceinline__ uint32_t bin_of(uint32_t key, uint32_t key_lo, uint32_t shift) {
    const uint32_t b = (key - key_lo) >> shift;
    return b < (uint32_t)kHistBins - 1u ? b : (uint32_t)kHistBins - 1u;
}

// exclusive prefix sum over the workgroup's threads; total returned through *total
template <int THREADS>
__device__ uint32_t cand_block_scan(uint32_t v, uint32_t *lds_wave /*[THREADS / 64]*/, uint32_t *total) {
    const uint32_t incl = wave_inclusive_scan(v);
    const int wave = threadIdx.x / kWave;
    __syncthreads();                       // lds_wave may still be in use by a previous scan
    if (lane_id() == kWave - 1) lds_wave[wave] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (int v2 = 0; v2 < THREADS / kWave; ++v2) {
        const uint32_t t = lds_wave[v2];
        if (v2 < wave) before += t;
        all += t;
    }
    *total = all;
    return before + incl - v;
}

__device__ void zero_global_hist(uint32_t *hist, int bins) {
    for (int i = threadIdx.x; i < bins; i += blockDim.x) hist[i] = 0u;
}

// ---------------------------------------------------------------- collect
// Where the sample's keys lie, by their 12 leading bits (s.hist): s.bin = the bin of the r-th largest, s.need = the number
// of samples in the bin of the mid-th largest.  1 <= mid <= r <= the number of samples.
__device__ void select_sample_bins(RowShared &s, uint32_t r, uint32_t mid) {
    constexpr int kPer = kBins1 / kBlk;                               // bins per thread, from the top
    uint32_t h[kPer], mine = 0u;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        h[j] = s.hist[kBins1 - 1 - ((int)threadIdx.x * kPer + j)];
        mine += h[j];
    }
    const uint32_t incl = wave_inclusive_scan(mine);
    const int wave = threadIdx.x / kWave;
    if (lane_id() == kWave - 1) s.wave_a[wave] = incl;
    __syncthreads();
    uint32_t run = incl - mine;
    for (int w = 0; w < wave; ++w) run += s.wave_a[w];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {                                  // each holds for one bin
        if (run < r && r <= run + h[j]) s.bin = (uint32_t)(kBins1 - 1 - ((int)threadIdx.x * kPer + j));
        if (run < mid && mid <= run + h[j]) s.need = h[j];
        run += h[j];
    }
    __syncthreads();
}

// Lower bound of the candidate keys and bin width from the sample, identical in every workgroup of a row (they depend on
// the data only).  key_lo: the lower edge of the bin, in a histogram of the keys' 12 leading bits (1/16 octave), that holds
// the sample's r-th largest key.  A finer bound would save a few per cent of the candidates, which cost little,
// for a second histogram pass, which costs a microsecond in every workgroup.  0 means "every entry is a candidate".
// shift: see widest_cold.
struct Guess {
    uint32_t key_lo, shift;
};
template <bool DIFF>
__device__ Guess guess_from_sample(RowShared &s, const float *a, const float *b, int64_t d, const SampleRule &rule) {
    static_assert(kBits2 + kBits3 == 19, "sample_rule counts samples in 2^19 keys");
    const int64_t ns = d < kSample ? d : kSample;
    if (rule.r > ns) return {0u, rule.widest};
    uint32_t skey[kSamplePer];
#pragma unroll
    for (int j = 0; j < kSamplePer; ++j) {
        const int64_t i = threadIdx.x + (int64_t)j * kBlk;
        skey[j] = 0xffffffffu;            // marks "no sample" (a magnitude key has bit 31 clear)
        if (i < ns) {
            int64_t e = i;
            if (d > kSample) e = ((i / kPieceLen) * (d - kPieceLen)) / (kPieces - 1) + (i % kPieceLen);
            skey[j] = mag_key(load_v<DIFF>(a, b, e));
        }
    }
    for (int i = threadIdx.x; i < kBins1; i += kBlk) s.hist[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSamplePer; ++j)
        if (skey[j] != 0xffffffffu) atomicAdd(&s.hist[skey[j] >> (kBits2 + kBits3)], 1u);
    __syncthreads();
    select_sample_bins(s, rule.r, rule.mid);
    const uint32_t near_t = s.need;
    const Guess g{s.bin << (kBits2 + kBits3), rule.widest - (near_t <= rule.most ? 0u : (near_t <= rule.most_next ? 1u : 2u))};
    __syncthreads();
    return g;
}

// Per-wavefront staging ring in LDS: candidates (position, value bits) are appended here and leave for the slot
// in global memory 64 at a time, as one full-width 8-byte store, instead of as many scattered stores.
constexpr uint32_t kRing = 128;              // entries of a staging ring (power of two, >= 128)
template <bool RESID>
struct StageRing {
    uint2 e[kRing];
    float r[RESID ? kRing : 1];
};
struct SlotOut {                             // a slot in global memory
    uint2 *cand;
    float *resid;
};

// What a wavefront needs to classify and count candidates.
struct CandFilter {
    uint32_t key_lo, shift;
    uint32_t *hist;          // the workgroup's LDS histogram
};

// Writes the entries [flushed, flushed + count) of the ring (count <= 64) to the slot and counts them into the
// histogram (here, with all lanes busy, rather than where they are found, a few lanes at a time).
template <bool RESID, class Ring>
__device__ __forceinline__ void ring_to_slot(const Ring &ring, uint32_t flushed, uint32_t count, int lane,
                                             const SlotOut &slot, const CandFilter &f) {
    if ((uint32_t)lane < count) {
        const uint2 rec = ring.e[(flushed + lane) & (kRing - 1)];
        slot.cand[flushed + lane] = rec;
        if constexpr (RESID) {
            if (slot.resid) slot.resid[flushed + lane] = ring.r[(flushed + lane) & (kRing - 1)];
        }
        atomicAdd(&f.hist[bin_of(rec.y & 0x7fffffffu, f.key_lo, f.shift)], 1u);
    }
}

// a - b = fl(a - b) + this, exactly (Knuth's two-sum; NaN where the difference is not finite)
__device__ __forceinline__ float rounding_of_difference(float a, float b) {
    const float x = a - b, b_seen = a - x, a_seen = x + b_seen;
    return (a - a_seen) + (b_seen - b);
}

// Appends the candidates among one step's entries (VEC per lane, lane-major order) to the slot.
// FULL: every entry of the step lies inside the piece, no bounds checks.
// RESID: v = fl(va - vb), and what the rounding took away goes along.
// cnt = candidates so far, flushed = how many of them are already in global memory (cnt - flushed < 64
// between calls; both are uniform over the wavefront).
template <int VEC, bool FULL, bool RESID, class Ring>
__device__ __forceinline__ void append_candidates(const float (&v)[VEC], const float (&va)[VEC], const float (&vb)[VEC],
                                                  int64_t e0, int64_t hi, const CandFilter &f, Ring &ring, int lane,
                                                  const SlotOut &slot, uint32_t &cnt, uint32_t &flushed) {
    bool c[VEC];
    uint32_t below = 0, all = 0;
#pragma unroll
    for (int t = 0; t < VEC; ++t) {
        c[t] = (FULL || e0 + t < hi) && mag_key(v[t]) >= f.key_lo;
        const uint64_t m = __ballot(c[t]);
        below += lanes_below(m);
        all += popc64(m);
    }
    if (all == 0) return;
    uint32_t pos = cnt + below;
    if (all > 64) {        // a dense step would not fit the ring: drain it, then store directly
        ring_to_slot<RESID>(ring, flushed, cnt - flushed, lane, slot, f);
#pragma unroll
        for (int t = 0; t < VEC; ++t) {
            if (c[t]) {
                slot.cand[pos] = make_uint2((uint32_t)(e0 + t), __float_as_uint(v[t]));
                if constexpr (RESID) {
                    if (slot.resid) slot.resid[pos] = rounding_of_difference(va[t], vb[t]);
                }
                atomicAdd(&f.hist[bin_of(mag_key(v[t]), f.key_lo, f.shift)], 1u);
                ++pos;
            }
        }
        cnt += all;
        flushed = cnt;
        return;
    }
#pragma unroll
    for (int t = 0; t < VEC; ++t) {
        if (c[t]) {
            ring.e[pos & (kRing - 1)] = make_uint2((uint32_t)(e0 + t), __float_as_uint(v[t]));
            if constexpr (RESID) ring.r[pos & (kRing - 1)] = rounding_of_difference(va[t], vb[t]);
            ++pos;
        }
    }
    cnt += all;
    if (cnt - flushed > kRing - 64) {        // keep room for the next step's candidates (at most 64)
        __builtin_amdgcn_wave_barrier();
        ring_to_slot<RESID>(ring, flushed, 64, lane, slot, f);
        flushed += 64;
    }
}

// Writes what is left in the ring at the end of a piece.
template <bool RESID, class Ring>
__device__ __forceinline__ void drain_ring(const Ring &ring, uint32_t flushed, uint32_t cnt, int lane,
                                           const SlotOut &slot, const CandFilter &f) {
    __builtin_amdgcn_wave_barrier();
    for (; flushed < cnt; flushed += 64)
        ring_to_slot<RESID>(ring, flushed, cnt - flushed < 64 ? cnt - flushed : 64, lane, slot, f);
}

// A wavefront walks its piece in steps of 256 entries, four per lane and load, kSteps steps per group.  Rows may start at
// any 4-byte address (rows of odd length: ef21_topk of 10 rows of 3000001, k = 30000, 52.5 us with 4-byte loads, 45 with 16-byte ones).
// Whole groups are loaded without any bounds check so that all loads of a group are in flight together; only the last
// piece of a row has a checked tail.
// MODE: kColdPass key_lo from the sample; kWarmPass from the threshold remembered in slot p.warm if there is
// one, else from the sample; kSecondPass: a row whose warm start failed, from the sample, into hist_b (in the count kernel).
// ADD != kNoAdd (kWarmPass): the rows are a + add_scale * add, written over a on the way.  A sample would find some entries of the row
// old and some new, so a row without a remembered threshold collects nothing here and is left to the count kernel.
// All kBlk threads of the workgroup must call; s and rings are the workgroup's.
template <bool DIFF, int MODE, bool RESID, int ADD, class Ring>
__device__ __forceinline__ void collect_rows(const TopkArgs &p, const Ws &w, RowShared &s, Ring (&rings)[kBlkWaves]) {
    const int64_t row = blockIdx.y, d = p.d;
    const float *a = p.a + row * d;
    static_assert(ADD == kNoAdd || (!DIFF && !RESID && MODE == kWarmPass), "see above");
    constexpr bool TWO = DIFF || ADD != kNoAdd;      // two arrays are read
    const float *b = DIFF ? p.b + row * d : (ADD ? p.add + row * d : nullptr);
    float *const out = ADD ? p.g_i + row * d : nullptr;
    RowInfo *info = w.info + row;
    CandFilter f;
    f.hist = s.hist;
    uint32_t *merged = w.hist_a + row * kHistBins;
    if constexpr (MODE == kSecondPass) {
        const Guess g = guess_from_sample<DIFF>(s, a, b, d, w.rule);
        f.key_lo = g.key_lo;
        f.shift = g.shift;
        merged = w.hist_b + row * kHistBins;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            info->key_lo2 = f.key_lo;
            info->shift2 = f.shift;
            info->use2 = 1u;
        }
    } else {
        uint32_t warm = 0u;                          // the remembered threshold's bin width
        if constexpr (MODE == kWarmPass) warm = info->warm_s[p.warm - 1];
        if (warm) {
            start_from(info->warm_T[p.warm - 1], warm, &f.key_lo, &f.shift);
        } else if constexpr (ADD) {
            f.key_lo = 0x80000000u;                  // above every key
            f.shift = w.rule.widest;
        } else {
            const Guess g = guess_from_sample<DIFF>(s, a, b, d, w.rule);
            f.key_lo = g.key_lo;
            f.shift = g.shift;
        }
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            info->key_lo = f.key_lo;
            info->shift = f.shift;
            info->use2 = 0u;
            info->ntie = 0u;                 // the count kernel appends to the list
            info->tie_min = 0xffffffffu;
            info->tie_max = 0u;
            info->warm_used = warm || ADD ? 1u : 0u;
            info->failed = kRowPending;
            info->arrived = 0u;
        }
    }
    for (int i = threadIdx.x; i < kHistBins; i += kBlk) s.hist[i] = 0u;
    __syncthreads();

    const int wave = wave_id(), lane = lane_id();
    const int64_t slot_no = (int64_t)blockIdx.x * kBlkWaves + wave;
    if (slot_no < w.nslot) {
        Ring &ring = rings[wave];
        const int64_t lo = slot_no * w.L;
        const int64_t hi = lo + w.L < d ? lo + w.L : d;
        const int64_t slot_at = (row * w.nslot + slot_no) * w.L;
        const SlotOut slot{w.cand + slot_at, RESID && w.resid ? w.resid + slot_at : nullptr};
        uint32_t cnt = 0, flushed = 0;
        constexpr int VEC = 4, kStep = kWave * VEC, kGroup = kStep * kSteps;
        int64_t base = lo;
        // Groups of kSteps steps, two register buffers: the next group's loads are issued before this group is
        // filtered, so that a wavefront has loads in flight while it computes.  After the last group the
        // "next" loads all read the piece's first 16 bytes (one cached line) instead of sitting behind a
        // branch.  What is in flight per compute unit is 1024 lanes x arrays x 2 kSteps x 16 bytes; measured best
        // at 64 to 128 KB (the C1 call, one array: 31.7 us with two steps, 36 with one, 33 with four).
        float4 va[kSteps], vb[kSteps];
        if (base + kGroup <= hi) {
#pragma unroll
            for (int u = 0; u < kSteps; ++u) {
                va[u] = stream_load4_any(a + base + u * kStep + lane * 4);
                if constexpr (TWO) vb[u] = stream_load4_any(b + base + u * kStep + lane * 4);
            }
        }
        for (; base + kGroup <= hi; base += kGroup) {
            const bool more = base + 2 * kGroup <= hi;
            float4 na[kSteps], nb[kSteps];
#pragma unroll
            for (int u = 0; u < kSteps; ++u) {
                const int64_t at = more ? base + kGroup + u * kStep + lane * 4 : lo;
                na[u] = stream_load4_any(a + at);
                if constexpr (TWO) nb[u] = stream_load4_any(b + at);
            }
#pragma unroll
            for (int u = 0; u < kSteps; ++u) {
                const float ea[VEC] = {va[u].x, va[u].y, va[u].z, va[u].w};
                float eb[VEC] = {}, v[VEC];
                if constexpr (TWO) {
                    eb[0] = vb[u].x; eb[1] = vb[u].y; eb[2] = vb[u].z; eb[3] = vb[u].w;
                }
#pragma unroll
                for (int t = 0; t < VEC; ++t) v[t] = DIFF ? ea[t] - eb[t] : (ADD ? fmaf(p.add_scale, eb[t], ea[t]) : ea[t]);
                if constexpr (ADD == kAddKept) store4_any(out + base + u * kStep + lane * 4, make_float4(v[0], v[1], v[2], v[3]));
                if constexpr (ADD == kAddStreamed) stream_store4_any(out + base + u * kStep + lane * 4, make_float4(v[0], v[1], v[2], v[3]));
                append_candidates<VEC, true, RESID>(v, ea, eb, base + u * kStep + lane * VEC, hi, f, ring, lane, slot, cnt, flushed);
            }
#pragma unroll
            for (int u = 0; u < kSteps; ++u) {
                va[u] = na[u];
                if constexpr (TWO) vb[u] = nb[u];
            }
        }
        if (base < hi) {                             // checked tail, less than a group, all loads issued first
            float ea[kSteps][VEC], eb[kSteps][VEC];
#pragma unroll
            for (int u = 0; u < kSteps; ++u)
#pragma unroll
                for (int t = 0; t < VEC; ++t) {
                    const int64_t e = base + u * kStep + lane * VEC + t;
                    ea[u][t] = e < hi ? a[e] : 0.f;
                    eb[u][t] = TWO && e < hi ? b[e] : 0.f;
                }
#pragma unroll
            for (int u = 0; u < kSteps; ++u) {
                float v[VEC];
#pragma unroll
                for (int t = 0; t < VEC; ++t) {
                    v[t] = DIFF ? ea[u][t] - eb[u][t] : (ADD ? fmaf(p.add_scale, eb[u][t], ea[u][t]) : ea[u][t]);
                    const int64_t e = base + u * kStep + lane * VEC + t;
                    if (ADD && e < hi) out[e] = v[t];
                }
                append_candidates<VEC, false, RESID>(v, ea[u], eb[u], base + u * kStep + lane * VEC, hi, f, ring, lane, slot, cnt, flushed);
            }
        }
        drain_ring<RESID>(ring, flushed, cnt, lane, slot, f);
        if (lane == 0) w.slot_cnt[row * w.nslot + slot_no] = cnt;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kHistBins; i += kBlk) {
        const uint32_t c = s.hist[i];
        if (c) atomicAdd(merged + i, c);
    }
}

template <bool DIFF, int MODE, int ADD = kNoAdd>
__global__ __launch_bounds__(kBlk) void split_collect_kernel(TopkArgs p, Ws w) {
    __shared__ RowShared s;
    __shared__ StageRing<false> rings[kBlkWaves];
    collect_rows<DIFF, MODE, false, ADD>(p, w, s, rings);
}

// ---------------------------------------------------------------- collect, two selections in one pass
// Algorithm 3 (EF21+) selects from two vectors built of the same arrays: the gradient s itself (line 5) and the
// difference s - g_i (line 6), and needs the squared norms of both (line 7).  This kernel reads s and g_i once
// and does the work of two collect passes and of the norm pass: candidates, histograms and slot counts of the
// difference go to workspace `wm` (arguments pm: a = s, b = g_i), those of s to workspace `wp` (warm-start memory
// warm_p), and every wavefront leaves (sum s^2, sum (s - g_i)^2) over its piece in norms[row][slot], the
// differences of the stored values taken exactly in fp64 and the sums in a fixed order.
template <bool WARM>
__global__ __launch_bounds__(kBlk) void split_collect_pair_kernel(TopkArgs pm, Ws wm, int warm_p, Ws wp,
                                                                  double2 *__restrict__ norms) {
    __shared__ RowShared s;                      // its histogram serves the sampling, then the difference
    __shared__ uint32_t hist_p[kHistBins];
    __shared__ StageRing<true> rings_m[kBlkWaves];
    __shared__ StageRing<false> rings_p[kBlkWaves];
    const int64_t row = blockIdx.y, d = pm.d;
    const float *a = pm.a + row * d, *b = pm.b + row * d;
    RowInfo *info_m = wm.info + row, *info_p = wp.info + row;
    CandFilter fm, fp;
    fm.hist = s.hist;
    fp.hist = hist_p;
    const uint32_t warm_m = WARM ? info_m->warm_s[pm.warm - 1] : 0u, warm_pl = WARM ? info_p->warm_s[warm_p - 1] : 0u;
    if (warm_m) {
        start_from(info_m->warm_T[pm.warm - 1], warm_m, &fm.key_lo, &fm.shift);
    } else {
        const Guess g = guess_from_sample<true>(s, a, b, d, wm.rule);
        fm.key_lo = g.key_lo;
        fm.shift = g.shift;
    }
    if (warm_pl) {
        start_from(info_p->warm_T[warm_p - 1], warm_pl, &fp.key_lo, &fp.shift);
    } else {
        const Guess g = guess_from_sample<false>(s, a, nullptr, d, wm.rule);
        fp.key_lo = g.key_lo;
        fp.shift = g.shift;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        info_m->key_lo = fm.key_lo; info_m->shift = fm.shift; info_m->use2 = 0u; info_m->ntie = 0u;
        info_m->tie_min = 0xffffffffu; info_m->tie_max = 0u;
        info_m->warm_used = warm_m ? 1u : 0u;
        info_m->failed = info_p->failed = kRowPending;
        info_m->arrived = info_p->arrived = 0u;
        info_p->key_lo = fp.key_lo; info_p->shift = fp.shift; info_p->use2 = 0u; info_p->ntie = 0u;
        info_p->tie_min = 0xffffffffu; info_p->tie_max = 0u;
        info_p->warm_used = warm_pl ? 1u : 0u;
    }
    for (int i = threadIdx.x; i < kHistBins; i += kBlk) {
        s.hist[i] = 0u;
        hist_p[i] = 0u;
    }
    __syncthreads();

    const int wave = wave_id(), lane = lane_id();
    const int64_t slot_no = (int64_t)blockIdx.x * kBlkWaves + wave;
    if (slot_no < wm.nslot) {
        StageRing<true> &ring_m = rings_m[wave];
        StageRing<false> &ring_p = rings_p[wave];
        const int64_t lo = slot_no * wm.L;
        const int64_t hi = lo + wm.L < d ? lo + wm.L : d;
        const int64_t slot_at = (row * wm.nslot + slot_no) * wm.L;           // the two layouts are the same
        const SlotOut slot_m{wm.cand + slot_at, wm.resid ? wm.resid + slot_at : nullptr};
        const SlotOut slot_p{wp.cand + slot_at, nullptr};
        uint32_t cnt_m = 0, flushed_m = 0, cnt_p = 0, flushed_p = 0;
        double sq_s = 0.0, sq_v = 0.0;
        constexpr int VEC = 4, kStep = kWave * VEC, kGroup = kStep * kSteps;
        int64_t base = lo;
        // one step of the wavefront: the squared norms of line 7, the difference of line 6, both filters
        auto filter_step = [&](const float (&vs)[VEC], const float (&vg)[VEC], int64_t e0, auto full) {
            float vd[VEC];
#pragma unroll
            for (int t = 0; t < VEC; ++t) {
                const double sv = (double)vs[t], dv = sv - (double)vg[t];            // exact
                sq_s += sv * sv;
                sq_v += dv * dv;
                vd[t] = vs[t] - vg[t];                                               // line 6: one fp32 subtraction
            }
            append_candidates<VEC, decltype(full)::value, false>(vs, vs, vs, e0, hi, fp, ring_p, lane, slot_p, cnt_p, flushed_p);
            append_candidates<VEC, decltype(full)::value, true>(vd, vs, vg, e0, hi, fm, ring_m, lane, slot_m, cnt_m, flushed_m);
        };
        // two register buffers, as in split_collect_kernel: the next group's loads before this group's work
        float4 va[kSteps], vb[kSteps];
        if (base + kGroup <= hi) {
#pragma unroll
            for (int u = 0; u < kSteps; ++u) {
                va[u] = stream_load4_any(a + base + u * kStep + lane * 4);
                vb[u] = stream_load4_any(b + base + u * kStep + lane * 4);
            }
        }
        for (; base + kGroup <= hi; base += kGroup) {
            const bool more = base + 2 * kGroup <= hi;
            float4 na[kSteps], nb[kSteps];
#pragma unroll
            for (int u = 0; u < kSteps; ++u) {
                const int64_t at = more ? base + kGroup + u * kStep + lane * 4 : lo;
                na[u] = stream_load4_any(a + at);
                nb[u] = stream_load4_any(b + at);
            }
#pragma unroll
            for (int u = 0; u < kSteps; ++u) {
                const float vs[VEC] = {va[u].x, va[u].y, va[u].z, va[u].w}, vg[VEC] = {vb[u].x, vb[u].y, vb[u].z, vb[u].w};
                filter_step(vs, vg, base + u * kStep + lane * VEC, std::true_type());
            }
#pragma unroll
            for (int u = 0; u < kSteps; ++u) {
                va[u] = na[u];
                vb[u] = nb[u];
            }
        }
        if (base < hi) {                             // checked tail, less than a group, all loads issued first
            float vs[kSteps][VEC], vg[kSteps][VEC];
#pragma unroll
            for (int u = 0; u < kSteps; ++u)
#pragma unroll
                for (int t = 0; t < VEC; ++t) {
                    const int64_t e = base + u * kStep + lane * VEC + t;
                    vs[u][t] = e < hi ? a[e] : 0.f;
                    vg[u][t] = e < hi ? b[e] : 0.f;
                }
#pragma unroll
            for (int u = 0; u < kSteps; ++u) filter_step(vs[u], vg[u], base + u * kStep + lane * VEC, std::false_type());
        }
        drain_ring<false>(ring_p, flushed_p, cnt_p, lane, slot_p, fp);
        drain_ring<true>(ring_m, flushed_m, cnt_m, lane, slot_m, fm);
        sq_s = wave_sum_f64(sq_s);
        sq_v = wave_sum_f64(sq_v);
        if (lane == 0) {
            wm.slot_cnt[row * wm.nslot + slot_no] = cnt_m;
            wp.slot_cnt[row * wp.nslot + slot_no] = cnt_p;
            norms[row * wm.nslot + slot_no] = make_double2(sq_s, sq_v);
        }
    }
    __syncthreads();
    uint32_t *merged_m = wm.hist_a + row * kHistBins, *merged_p = wp.hist_a + row * kHistBins;
    for (int i = threadIdx.x; i < kHistBins; i += kBlk) {
        const uint32_t cm = s.hist[i], cp = hist_p[i];
        if (cm) atomicAdd(merged_m + i, cm);
        if (cp) atomicAdd(merged_p + i, cp);
    }
}

// ---------------------------------------------------------------- count
// The exact one-workgroup algorithm on the original data for a row whose guess failed, and the message index of
// the row if the caller asked for one.  All kCandThreads threads of the workgroup must call.
// The threshold found is remembered as any other, so that the row's next call does not start from a sample again, with
// next_shift as the bin width.
// SUMS (Algorithm 3): the whole row's sum of kept squares goes to its first slot, the others' are zero.
template <bool DIFF, int UPDATE, bool SUMS>
__device__ void rescue_row(RowShared &rs, const TopkArgs &p, const Ws &w, int64_t row, uint32_t next_shift) {
    row_topk<DIFF, UPDATE>(rs, p, row);
    if (p.warm > 0) {
        uint32_t *part = rs.hist, T = 0xffffffffu;
        __syncthreads();                    // the pairs are written, the histogram is done with
        for (int64_t at = threadIdx.x; at < p.k; at += kCandThreads) {
            const uint32_t key = mag_key(p.out_val[row * p.k + at]);
            T = key < T ? key : T;
        }
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) {
            const uint32_t other = __shfl_xor(T, o, kWave);
            T = other < T ? other : T;
        }
        if (lane_id() == 0) part[threadIdx.x / kWave] = T;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int v = 0; v < kCandWaves; ++v) T = part[v] < T ? part[v] : T;
            w.info[row].warm_T[p.warm - 1] = T;
            w.info[row].warm_s[p.warm - 1] = next_shift;
        }
    }
    if constexpr (SUMS) {
        static_assert(UPDATE == kNoUpdate, "the vectors still hold what was selected from");
        double *part = reinterpret_cast<double *>(rs.hist);
        __syncthreads();                    // the pairs are written, rs.hist is done with
        double sq = 0.0;
        for (int64_t at = threadIdx.x; at < p.k; at += kCandThreads) {
            const int64_t e = row * p.d + p.out_idx[row * p.k + at];
            const double v = (double)p.a[e] - (DIFF ? (double)p.b[e] : 0.0);
            sq += v * v;
        }
        sq = wave_sum_f64(sq);
        if (lane_id() == 0) part[threadIdx.x / kWave] = sq;
        __syncthreads();
        double all = 0.0;
        for (int v = 0; v < kCandWaves; ++v) all += part[v];
        for (int64_t t = threadIdx.x; t < w.nslot; t += kCandThreads) w.kept[row * w.nslot + t] = t == 0 ? all : 0.0;
    }
    if (p.agg_start) {                  // from the pairs just written
        __syncthreads();
        const int32_t *out = p.out_idx + row * p.k;
        int32_t *start = p.agg_start + row * (p.agg_nblk + 1);
        for (int64_t at = threadIdx.x; at < p.k; at += kCandThreads) {
            const int64_t b_cur = out[at] >> p.agg_shift;
            const int64_t b_prev = at > 0 ? out[at - 1] >> p.agg_shift : -1;
            for (int64_t b = b_prev + 1; b <= b_cur; ++b) start[b] = (int32_t)at;
            if (at == p.k - 1)
                for (int64_t b = b_cur + 1; b <= p.agg_nblk; ++b) start[b] = (int32_t)p.k;
        }
    }
}

// A wavefront of the count and emit kernels takes one slot.  The first kPre steps of 64 candidates (clamped to the
// slot's capacity, a multiple of 512) are loaded at the very start of the kernel, together
// with everything else whose address does not depend on the prologue, so that a workgroup waits for memory once,
// not once per step of its prologue.  See cand_steps for kPre.

// Grid (slot blocks, n).  Prologue of every workgroup: T's bin from the row's histogram, and whether the row failed (see
// the head of the file); the row's first workgroup then selects it by the exact one-workgroup algorithm on the original
// data (DIFF and UPDATE matter here only).  Otherwise a slot's candidates in bins above T's are counted, those in T's bin
// go to the tie list.  (An extra workgroup per row for the exact algorithm, as there used to be, keeps a compute unit from
// the last of 255 others for a few microseconds, here and in the emit kernel, since a unit holds one of them: step of
// n = 15, d = 5 million, k = 50000 10.1 and 40.6 us in the two kernels, 6.7 and 31.7 without.)
//
// A row whose warm start failed is collected again from the sample instead, by all its workgroups, into hist_b; the one that is done last looks
// for T's bin in it and says what it is, and then all that are still there count the slots, a block of them at a time.  Nobody has to be
// there: a workgroup waits for the bin for kPatience at most and then ends, and what the others have not taken the last one counts.
// Where every row's guess fails at every step (differences a thousand times larger and smaller in turn), us a step by itself, as a launch of its own and
// here: n = 8, d = 10^5, k = 3000 43 and 46; n = 8, d = 10^6, k = 10^4 80 and 80; n = 4, d = 3 million, k = 200 000 132 and 131; n = 8, d = 11.2 million,
// k = 112 000 587 and 493; n = 1, d = 12 million, k = 77 000 136 and 138.  With the row's slots counted by the last workgroup alone, one after the other, n =
// 4, d = 3 million took 243, and differences that shrink to three fifths from step to step, n = 1, d = 8 million, k = 60 000, 304 against 96.
// (As a launch of its own, which nearly always ended at once, the second pass took 3.8 to 4.6 us of
// every warm call: n = 8, d = 10^5, k = 3000 26.6 us a step with it, 24.5 so; n = 8, d = 10^6, k = 10^4 38.7 and 36.2; EF on n = 5, d = 10^6, k =
// 50 000 44.4 and 42.1; EF21+ on n = 5, d = 10^6 55.2 and 53.0.)
constexpr uint64_t kPatience = 2000;             // of the clock's 100 MHz: 20 us, some times what the last one is late by
struct CountShared {
    RowShared rs;
    uint32_t wave[kCandWaves], out[4], last;
};
// The bin of the row's histogram that holds the need-th largest key: the largest bin b with count(bins > b) < need <= count(bins >= b),
// from the thread's bins h, the highest first.  out[0] = b, out[1] = need - count(bins > b), out[2] = the bin's entries; false if there
// are fewer than `need`.  All threads of the workgroup must call.
constexpr int kPerThread = kHistBins / kCandThreads;
__device__ __forceinline__ bool threshold_bin(const uint32_t (&h)[kPerThread], uint32_t need, uint32_t (&lds_wave)[kCandWaves],
                                              uint32_t (&out)[4]) {
    uint32_t mine = 0, total;
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) mine += h[j];
    const uint32_t higher = cand_block_scan<kCandThreads>(mine, lds_wave, &total);
    if (higher < need && need <= higher + mine) {         // exactly one thread, if total >= need
        uint32_t run = higher;
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) {
            if (need > run && need <= run + h[j]) {
                out[0] = (uint32_t)(kHistBins - 1 - ((int)threadIdx.x * kPerThread + j));
                out[1] = need - run;
                out[2] = h[j];
            }
            run += h[j];
        }
    }
    __syncthreads();
    return total >= need;
}
template <bool DIFF, int UPDATE, int kPre, bool SUMS>
__device__ __forceinline__ void count_rows(const TopkArgs &p, const Ws &w, CountShared &sh, StageRing<DIFF && SUMS> (&rings)[kBlkWaves]) {
    RowShared &rs = sh.rs;
    uint32_t (&lds_wave)[kCandWaves] = sh.wave, (&lds_out)[4] = sh.out;
    const int64_t row = blockIdx.y;
    const int tid = threadIdx.x, wave = wave_id(), lane = lane_id();
    RowInfo *info = w.info + row;
    const int64_t slot_no = (int64_t)blockIdx.x * kCandWaves + wave;
    // everything whose address is known now
    const RowInfo ri = *info;
    uint32_t h[kPerThread];
#pragma unroll
    for (int j = 0; j < kPerThread; ++j) h[j] = w.hist_a[row * kHistBins + kHistBins - 1 - (tid * kPerThread + j)];
    uint2 c[kPre];
    const bool active = slot_no < w.nslot;
    const int64_t slc = active ? slot_no : 0;
    uint32_t cnt = w.slot_cnt[row * w.nslot + slc];
    const uint2 *slot = w.cand + (row * w.nslot + slc) * w.L;
#pragma unroll
    for (int q = 0; q < kPre; ++q) c[q] = slot[q * kWave + lane];
    if (!active) cnt = 0u;

    uint32_t key_lo = ri.key_lo, shift = ri.shift, bin_a = 0, need_a = 0;
    bool crowded = false;
    auto find_bin = [&]() {                      // false: fewer than k candidates, or T beyond the window
        const bool enough = threshold_bin(h, (uint32_t)p.k, lds_wave, lds_out);
        bin_a = enough ? lds_out[0] : 0u;
        need_a = enough ? lds_out[1] : 0u;
        const bool found = enough && bin_a != (uint32_t)kHistBins - 1u;
        crowded = found && lds_out[2] > (uint32_t)kTieCap;             // too many to list: see RowInfo::tie_min
        return found;
    };
    auto state = [&](bool found) { return found ? (crowded ? kRowCrowded : kRowFine) : kRowFailed; };
    const bool found = find_bin(), again = !found && ri.warm_used != 0u;
    if (again) {
        __syncthreads();                         // lds_out has been read
        collect_rows<DIFF, kSecondPass, DIFF && SUMS, kNoAdd>(p, w, rs, rings);
        if (draw_ticket(&info->arrived, gridDim.x, &sh.last)) {
            key_lo = info->key_lo2;
            shift = info->shift2;
#pragma unroll
            for (int j = 0; j < kPerThread; ++j) {
                uint32_t *bin = w.hist_b + row * kHistBins + kHistBins - 1 - (tid * kPerThread + j);
                h[j] = *bin;
                *bin = 0u;                       // consumed: zero for the next time
            }
            const bool found_now = find_bin();
            if (tid == 0) {
                info->bin_a = bin_a;
                info->need_a = need_a;
                __hip_atomic_store(&info->failed, (uint32_t)state(found_now), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (!found_now) {
                rescue_row<DIFF, UPDATE, SUMS>(rs, p, w, row, widest_warm(p.k, p.d));
                return;
            }
        } else {
            if (tid == 0) {
                const uint64_t since = wall_clock64();
                uint32_t now;
                while ((now = __hip_atomic_load(&info->failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == kRowPending &&
                       wall_clock64() - since < kPatience)
                    __builtin_amdgcn_s_sleep(4);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                lds_out[3] = now;
            }
            __syncthreads();
            const uint32_t now = lds_out[3];
            if (now == kRowPending || now == kRowFailed) return;
            key_lo = info->key_lo2;
            shift = info->shift2;
            bin_a = info->bin_a;
            crowded = now == kRowCrowded;
        }
    } else {
        if (blockIdx.x == 0 && tid == 0) {
            info->failed = state(found);
            info->bin_a = bin_a;
            info->need_a = need_a;
        }
        if (!found) {
            if (blockIdx.x == 0) rescue_row<DIFF, UPDATE, SUMS>(rs, p, w, row, widest_warm(p.k, p.d));
            return;
        }
    }
    uint2 *tie = w.tie + row * kTieCap;
    uint32_t key_min = 0xffffffffu, key_max = 0u;
    for (int64_t s = slot_no;;) {                // this wavefront's slot, or those of the blocks that the workgroup takes
        if (again) {
            __syncthreads();                     // lds_out[3] has been read
            if (tid == 0) lds_out[3] = atomicAdd(&info->arrived, 1u) - gridDim.x;
            __syncthreads();
            const uint32_t block = lds_out[3];
            if (block >= gridDim.x) break;
            s = (int64_t)block * kCandWaves + wave;
            cnt = s < w.nslot ? w.slot_cnt[row * w.nslot + s] : 0u;
            slot = w.cand + (row * w.nslot + (s < w.nslot ? s : 0)) * w.L;
        }
        uint32_t above = 0, inbin = 0;
        for (uint32_t j0 = 0; j0 < cnt; j0 += kWave * kPre) {
            if (j0 > 0 || again) {
#pragma unroll
                for (int q = 0; q < kPre; ++q) {
                    const uint32_t j = j0 + q * kWave + lane;
                    c[q] = slot[j < cnt ? j : 0u];           // clamped: no load behind a branch
                }
            }
#pragma unroll
            for (int q = 0; q < kPre; ++q) {
                const uint32_t j = j0 + q * kWave + lane;
                const uint32_t key = c[q].y & 0x7fffffffu;
                const uint32_t bin = bin_of(key < key_lo ? key_lo : key, key_lo, shift);
                above += popc64(__ballot(j < cnt && bin > bin_a));
                const bool in_bin = j < cnt && bin == bin_a;
                if (!crowded) {
                    const uint32_t at = wave_append(in_bin, &info->ntie);
                    if (in_bin && at < (uint32_t)kTieCap) tie[at] = make_uint2(c[q].x, key);
                } else {
                    inbin += popc64(__ballot(in_bin));
                    key_min = in_bin && key < key_min ? key : key_min;
                    key_max = in_bin && key > key_max ? key : key_max;
                }
            }
        }
        if (lane == 0 && s < w.nslot) {
            w.slot_above[row * w.nslot + s] = above;
            if (crowded) w.slot_inbin[row * w.nslot + s] = inbin;
        }
        if (!again) break;
    }
    if (crowded) {
#pragma unroll
        for (int o = kWave / 2; o > 0; o >>= 1) {
            const uint32_t lo_o = __shfl_xor(key_min, o, kWave), hi_o = __shfl_xor(key_max, o, kWave);
            key_min = lo_o < key_min ? lo_o : key_min;
            key_max = hi_o > key_max ? hi_o : key_max;
        }
        if (lane == 0 && key_min <= key_max) {
            atomicMin(&info->tie_min, key_min);
            atomicMax(&info->tie_max, key_max);
        }
    }
}

template <bool DIFF, int UPDATE, int kPre>
__global__ __launch_bounds__(kCandThreads) void cand_count_kernel(TopkArgs p, Ws w) {
    __shared__ CountShared sh;
    __shared__ StageRing<false> rings[kBlkWaves];
    count_rows<DIFF, UPDATE, kPre, false>(p, w, sh, rings);
}

// The two selections of Algorithm 3 in one launch: grid (.., n, 2).  (Likewise cand_emit_pair_kernel.)
template <int kPre>
__global__ __launch_bounds__(kCandThreads) void cand_count_pair_kernel(TopkArgs pp, Ws wp, TopkArgs pm, Ws wm) {
    __shared__ CountShared sh;
    __shared__ union {
        StageRing<false> plain[kBlkWaves];
        StageRing<true> markov[kBlkWaves];
    } rings;
    if (blockIdx.z == 0) count_rows<false, kNoUpdate, kPre, true>(pp, wp, sh, rings.plain);
    else count_rows<true, kNoUpdate, kPre, true>(pm, wm, sh, rings.markov);
}

// Ordered emission by one wavefront that walks candidates in position order, 64 at a time: the running output
// offset, the ties seen so far, and (if asked for) the aggregation's message index, start[b] = output position of
// the first kept entry at or beyond coordinate b << shift.  A wavefront's span [span_lo, span_end) is a whole number
// of index blocks, so every block begins inside exactly one wavefront's span, and that wavefront writes its start:
// when it keeps the first entry at or beyond the block's first coordinate, or at the end of its span for the
// blocks that follow its last kept entry (all of them if it kept nothing).
template <bool DIFF, int UPDATE, bool SUMS>
struct Emitter {
    const TopkArgs &p;
    int64_t row;
    uint32_t T, q;               // threshold key; entries equal to T that are kept (the first q in position order)
    uint32_t out_run, eq_run;    // kept entries, and entries equal to T, before the next step
    int32_t *out_idx;
    float *out_val;
    int32_t *agg_start;
    int64_t last_b;              // index blocks up to here have their start
    int lane;
    double kept_sq = 0.0;        // SUMS: this lane's kept entries, unrounded and squared

    __device__ Emitter(const TopkArgs &p_, int64_t row_, uint32_t T_, uint32_t q_, uint32_t gt_before,
                       uint32_t eq_before, int64_t span_lo, int lane_)
        : p(p_), row(row_), T(T_), q(q_), out_run(gt_before + (eq_before < q_ ? eq_before : q_)), eq_run(eq_before),
          out_idx(p_.out_idx + row_ * p_.k), out_val(p_.out_val + row_ * p_.k),
          agg_start(p_.agg_start ? p_.agg_start + row_ * (p_.agg_nblk + 1) : nullptr),
          last_b((span_lo >> p_.agg_shift) - 1), lane(lane_) {}

    // one step: `in` marks the lanes that hold a candidate (position rec.x, value bits rec.y); all lanes call.
    // have_b: b_pre is the value of b at the candidate's position, loaded by the caller beforehand.  resid (SUMS of a
    // difference): what its rounding took away; not finite: the difference is formed again.
    __device__ __forceinline__ void step(bool in, uint2 rec, bool have_b = false, float b_pre = 0.f, float resid = 0.f) {
        const uint32_t key = rec.y & 0x7fffffffu;
        const bool gt = in && key > T, eq = in && key == T;
        const uint64_t m_gt = __ballot(gt), m_eq = __ballot(eq);
        const uint32_t eq_below = eq_run + lanes_below(m_eq);
        const uint32_t ties_before = (eq_below < q ? eq_below : q) - (eq_run < q ? eq_run : q);
        const bool keep = gt || (eq && eq_below < q);
        const uint32_t pos = out_run + lanes_below(m_gt) + ties_before;
        if (keep) {
            const float v = __uint_as_float(rec.y);
            out_idx[pos] = (int32_t)rec.x;
            out_val[pos] = v;
            const int64_t at = row * p.d + (int64_t)rec.x;
            if constexpr (UPDATE == kAddUpdate) p.g_i[at] = (have_b ? b_pre : p.b[at]) + v;      // Algorithm 2, line 6
            if constexpr (UPDATE == kClearUpdate) p.g_i[at] = 0.f;                               // Algorithm 4
            if constexpr (SUMS) {
                double exact = (double)v;
                if constexpr (DIFF)
                    exact = fabsf(resid) <= 3.0e38f ? exact + (double)resid : (double)p.a[at] - (double)p.b[at];
                kept_sq += exact * exact;
            }
        }
        if (agg_start) {
            const uint64_t m_keep = __ballot(keep);
            if (m_keep) {
                const int64_t b_cur = (int64_t)(rec.x >> p.agg_shift);
                const uint64_t lower = m_keep & ((1ull << lane) - 1ull);
                const int prev_lane = lower ? 63 - __clzll((long long)lower) : 0;
                const int64_t b_before = __shfl(b_cur, prev_lane, kWave);
                const int64_t b_prev = lower ? b_before : last_b;
                if (keep)
                    for (int64_t b = b_prev + 1; b <= b_cur; ++b) agg_start[b] = (int32_t)pos;
                last_b = __shfl(b_cur, 63 - __clzll((long long)m_keep), kWave);
            }
        }
        const uint32_t eq_next = eq_run + popc64(m_eq);
        out_run += popc64(m_gt) + ((eq_next < q ? eq_next : q) - (eq_run < q ? eq_run : q));
        eq_run = eq_next;
    }

    // after the last step of a span that ends at span_end (clamped to the row's end by the caller)
    __device__ __forceinline__ void finish(int64_t span_end) {
        if (!agg_start) return;
        const int64_t b_last = ((span_end - 1) >> p.agg_shift) + (span_end == p.d ? 1 : 0);   // the row's end: start[nblk]
        for (int64_t b = last_b + 1 + lane; b <= b_last; b += kWave) agg_start[b] = (int32_t)out_run;
    }
};

// ---------------------------------------------------------------- emit
// Ordered emission.  Prologue of every workgroup: the tie list ranked (larger key first, lower position first
// among equal keys): the entry that need_a - 1 others precede is the last one kept, its key is T, and q counts it
// and the equal keys before it.  The output offset of a slot is the number of kept entries in all earlier slots:
// their candidates above T's bin (slot_above, summed by the workgroup) plus the listed entries before the slot's
// first position that are kept.  Grid (slot blocks, n); a row whose crowded bin (see RowInfo::tie_min) turned out to hold
// different keys is selected by its first workgroup, by the exact algorithm.  A crowded bin of equal keys needs no
// list: T is that key, and the ties before a slot are the earlier slots' entries of the bin (slot_inbin).
// SUMS (Algorithm 3): the sum of the kept squares of every slot goes to w.kept.
struct EmitShared {
    RowShared rs;                                // the rescue's
    uint32_t before_above[kCandWaves], own_above[kCandWaves], before_inbin[kCandWaves], own_inbin[kCandWaves];
    uint32_t tie_key[kTieCap], tie_idx[kTieCap];
    uint32_t T, q;
};
template <bool DIFF, int UPDATE, int kPre, bool SUMS>
__device__ __forceinline__ void emit_rows(const TopkArgs &p, const Ws &w, EmitShared &sh) {
    RowShared &rs = sh.rs;
    uint32_t (&before_above)[kCandWaves] = sh.before_above, (&own_above)[kCandWaves] = sh.own_above;
    uint32_t (&before_inbin)[kCandWaves] = sh.before_inbin, (&own_inbin)[kCandWaves] = sh.own_inbin;
    uint32_t (&tie_key)[kTieCap] = sh.tie_key, (&tie_idx)[kTieCap] = sh.tie_idx;
    uint32_t &sh_T = sh.T, &sh_q = sh.q;
    static_assert(kTieCap <= kCandThreads, "one listed entry per thread");
    const int64_t row = blockIdx.y;
    const int tid = threadIdx.x, wave = wave_id(), lane = lane_id();
    RowInfo *info = w.info + row;
    const int64_t sl0 = (int64_t)blockIdx.x * kCandWaves, slot_no = sl0 + wave;
    // everything whose address is known now
    const RowInfo ri = *info;
    const bool crowded = ri.failed == kRowCrowded;
    const uint2 listed = w.tie[row * kTieCap + (tid < kTieCap ? tid : 0)];
    const uint32_t *slot_above = w.slot_above + row * w.nslot;
    const uint32_t *slot_inbin = w.slot_inbin + row * w.nslot;
    uint32_t part = 0, part_in = 0;
    for (int64_t t = tid; t < sl0; t += kCandThreads) {
        part += slot_above[t];
        if (crowded) part_in += slot_inbin[t];
    }
    uint2 c[kPre];
    const bool active = slot_no < w.nslot;
    const int64_t slc = active ? slot_no : 0;
    const uint32_t mine = active ? slot_above[slc] : 0u;
    const uint32_t mine_in = active && crowded ? slot_inbin[slc] : 0u;
    uint32_t cnt = w.slot_cnt[row * w.nslot + slc];
    const uint2 *slot = w.cand + (row * w.nslot + slc) * w.L;
#pragma unroll
    for (int q = 0; q < kPre; ++q) c[q] = slot[q * kWave + lane];
    if (!active) cnt = 0u;
    // Line 6 needs g_i at the kept positions, scattered over the row: the loads for the wavefront's first
    // candidates that can be kept (those in T's bin or above: T itself is not known yet) are issued here, with
    // everything else, instead of one step at a time between the stores of the emission.
    float bpre[kPre], resid[kPre];
    if constexpr (DIFF && SUMS) {
#pragma unroll
        for (int q = 0; q < kPre; ++q)
            resid[q] = w.resid ? w.resid[slot - w.cand + q * kWave + lane] : INFINITY;
    }
    if constexpr (UPDATE == kAddUpdate) {
        const uint32_t key_lo = ri.use2 != 0u ? ri.key_lo2 : ri.key_lo, shift = ri.use2 != 0u ? ri.shift2 : ri.shift;
#pragma unroll
        for (int q = 0; q < kPre; ++q) {
            const uint32_t key = c[q].y & 0x7fffffffu;
            const bool have = (uint32_t)(q * kWave + lane) < cnt &&
                              bin_of(key < key_lo ? key_lo : key, key_lo, shift) >= ri.bin_a;
            bpre[q] = p.b[row * p.d + (have ? (int64_t)c[q].x : 0)];
        }
    }

    if (blockIdx.x == 0) zero_global_hist(w.hist_a + row * kHistBins, kHistBins);        // consumed: zero for the next call
    if (ri.failed == kRowFailed) return;         // the whole workgroup
    if (crowded && ri.tie_min != ri.tie_max) {
        if (blockIdx.x == 0) rescue_row<DIFF, UPDATE, SUMS>(rs, p, w, row, warm_shift(p.k, p.d, kCrowdedBin, 0u));
        return;
    }
    const uint32_t ntie = crowded ? 0u : (ri.ntie < (uint32_t)kTieCap ? ri.ntie : (uint32_t)kTieCap);
    const uint32_t my_idx = listed.x, my_key = listed.y;
    if ((uint32_t)tid < ntie) {
        tie_idx[tid] = my_idx;
        tie_key[tid] = my_key;
    }
    __syncthreads();
    if ((uint32_t)tid < ntie) {
        uint32_t larger = 0, equal_before = 0;
        for (uint32_t j = 0; j < ntie; ++j) {
            const uint32_t kj = tie_key[j], ij = tie_idx[j];
            larger += kj > my_key ? 1u : 0u;
            equal_before += (kj == my_key && ij < my_idx) ? 1u : 0u;
        }
        if (larger + equal_before == ri.need_a - 1u) {       // exactly one thread
            sh_T = my_key;
            sh_q = equal_before + 1u;
        }
    }
    __syncthreads();
    const uint32_t T = crowded ? ri.tie_min : sh_T, q = crowded ? ri.need_a : sh_q;
    if (blockIdx.x == 0 && tid == 0) {
        const int mem = p.warm > 0 ? p.warm - 1 : 0;
        static_assert(kWarmSlots == 1, "mem is zero; as an index it would put ri into scratch memory");
        info->warm_T[mem] = T;
        info->warm_s[mem] = p.warm > 0 ? warm_start(p.k, p.d, crowded, ntie, ri.use2 != 0u ? ri.shift2 : ri.shift,
                                                    ri.warm_s[0] != 0u, ri.warm_T[0], T, UPDATE == kClearUpdate) : 0u;
    }

    part = wave_sum_u32(part);
    part_in = wave_sum_u32(part_in);
    // listed entries before this wavefront's first position: kept ones above T, and ties
    const uint32_t my_lo = (uint32_t)(slot_no * w.L);
    uint32_t list_gt = 0, list_eq = 0;
    for (uint32_t j = lane; j < ntie; j += kWave) {
        const uint32_t kj = tie_key[j];
        if (tie_idx[j] < my_lo) {
            list_gt += kj > T ? 1u : 0u;
            list_eq += kj == T ? 1u : 0u;
        }
    }
    list_gt = wave_sum_u32(list_gt);
    list_eq = wave_sum_u32(list_eq);
    if (lane == 0) {
        before_above[wave] = part;
        own_above[wave] = mine;
        before_inbin[wave] = part_in;
        own_inbin[wave] = mine_in;
    }
    __syncthreads();
    if (slot_no >= w.nslot) return;
    uint32_t gt_run = list_gt, eq_run = list_eq;
    for (int v = 0; v < kCandWaves; ++v) {
        gt_run += before_above[v] + (v < wave ? own_above[v] : 0u);
        eq_run += before_inbin[v] + (v < wave ? own_inbin[v] : 0u);      // zero unless the bin is crowded
    }
    Emitter<DIFF, UPDATE, SUMS> em(p, row, T, q, gt_run, eq_run, slot_no * w.L, lane);
    for (uint32_t j0 = 0; j0 < cnt; j0 += kWave * kPre) {
        if (j0 > 0) {
#pragma unroll
            for (int u = 0; u < kPre; ++u) {
                const uint32_t j = j0 + u * kWave + lane;
                c[u] = slot[j < cnt ? j : 0u];           // clamped: no load behind a branch
                if constexpr (DIFF && SUMS)
                    resid[u] = w.resid ? w.resid[slot - w.cand + (j < cnt ? j : 0u)] : INFINITY;
            }
        }
#pragma unroll
        for (int u = 0; u < kPre; ++u) {
            if constexpr (DIFF && SUMS) em.step(j0 + u * kWave + lane < cnt, c[u], false, 0.f, resid[u]);
            else if constexpr (UPDATE == kAddUpdate) em.step(j0 + u * kWave + lane < cnt, c[u], j0 == 0, bpre[u]);
            else em.step(j0 + u * kWave + lane < cnt, c[u]);
        }
    }
    if constexpr (SUMS) {
        const double sq = wave_sum_f64(em.kept_sq);
        if (lane == 0 && slot_no < w.nslot) w.kept[row * w.nslot + slot_no] = sq;
    }
    const int64_t span_end = (slot_no + 1) * w.L;
    em.finish(span_end < p.d ? span_end : p.d);
}

template <bool DIFF, int UPDATE, int kPre>
__global__ __launch_bounds__(kCandThreads) void cand_emit_kernel(TopkArgs p, Ws w) {
    __shared__ EmitShared sh;
    emit_rows<DIFF, UPDATE, kPre, false>(p, w, sh);
}

template <int kPre>
__global__ __launch_bounds__(kCandThreads) void cand_emit_pair_kernel(TopkArgs pp, Ws wp, TopkArgs pm, Ws wm) {
    __shared__ EmitShared sh;
    if (blockIdx.z == 0) emit_rows<false, kNoUpdate, kPre, true>(pp, wp, sh);
    else emit_rows<true, kNoUpdate, kPre, true>(pm, wm, sh);
}

__global__ __launch_bounds__(kCandThreads) void zero_words_kernel(uint32_t *p, size_t words) {
    const size_t stride = (size_t)gridDim.x * kCandThreads;
    for (size_t i = (size_t)blockIdx.x * kCandThreads + threadIdx.x; i < words; i += stride) p[i] = 0u;
}

void launch_collect(const TopkArgs &p, const Ws &w, hipStream_t stream) {
    const dim3 grid((unsigned)w.G, (unsigned)p.n), block(kBlk);
    const bool diff = p.b != nullptr, warm = p.warm > 0;
    if (diff && warm) hipLaunchKernelGGL((split_collect_kernel<true, kWarmPass>), grid, block, 0, stream, p, w);
    else if (diff) hipLaunchKernelGGL((split_collect_kernel<true, kColdPass>), grid, block, 0, stream, p, w);
    else if (warm) hipLaunchKernelGGL((split_collect_kernel<false, kWarmPass>), grid, block, 0, stream, p, w);
    else hipLaunchKernelGGL((split_collect_kernel<false, kColdPass>), grid, block, 0, stream, p, w);
}

// ---------------------------------------------------------------- k = 1: the entry of largest magnitude
// Top-1 (the compressor of the paper's first experiment) needs no threshold and no candidates: every thread
// keeps the best entry of its share as one 64-bit word, key << 32 | ~position (a larger word = a larger
// magnitude, or the same magnitude at a lower position), the words are reduced over the wavefront and the
// workgroup, and one 64-bit atomic maximum per workgroup lands in the row's slot (the first two words of the
// row's histogram in the workspace, which are zero between calls).  A second, tiny kernel turns the slot into
// the message, applies line 6 and clears the slot.
constexpr int kArgThreads = 256, kArgWaves = kArgThreads / kWave;

template <bool DIFF>
__global__ __launch_bounds__(kArgThreads) void argmax_stream_kernel(TopkArgs p, Ws w, int64_t piece) {
    __shared__ unsigned long long best_of_wave[kArgWaves];
    const int64_t row = blockIdx.y, d = p.d;
    const float *a = p.a + row * d;
    const float *b = DIFF ? p.b + row * d : nullptr;
    const int64_t lo = (int64_t)blockIdx.x * piece, hi = lo + piece < d ? lo + piece : d;
    unsigned long long best = 0ull;
    auto see = [&](float v, int64_t e) {
        const unsigned long long word = ((unsigned long long)mag_key(v) << 32) | (0xffffffffu - (uint32_t)e);
        best = word > best ? word : best;
    };
    constexpr int kUnroll = DIFF ? 4 : 8;
    constexpr int64_t kStep = (int64_t)kArgThreads * 4;
    int64_t e = lo + (int64_t)threadIdx.x * 4;                   // rows may start at any 4-byte address
    for (; e + (kUnroll - 1) * kStep + 4 <= hi; e += kUnroll * kStep) {
        float4 va[kUnroll], vb[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            va[u] = stream_load4_any(a + e + u * kStep);
            if constexpr (DIFF) vb[u] = stream_load4_any(b + e + u * kStep);
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if constexpr (DIFF) {
                va[u].x -= vb[u].x;
                va[u].y -= vb[u].y;
                va[u].z -= vb[u].z;
                va[u].w -= vb[u].w;
            }
            const int64_t e0 = e + u * kStep;
            see(va[u].x, e0);
            see(va[u].y, e0 + 1);
            see(va[u].z, e0 + 2);
            see(va[u].w, e0 + 3);
        }
    }
    for (; e + 4 <= hi; e += kStep) {
        float4 va = stream_load4_any(a + e);
        if constexpr (DIFF) {
            const float4 vb = stream_load4_any(b + e);
            va.x -= vb.x;
            va.y -= vb.y;
            va.z -= vb.z;
            va.w -= vb.w;
        }
        see(va.x, e);
        see(va.y, e + 1);
        see(va.z, e + 2);
        see(va.w, e + 3);
    }
    for (; e < hi; ++e) see(load_v<DIFF>(a, b, e), e);           // one thread: the last entries of a row of odd length
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const unsigned long long other = __shfl_xor(best, o, kWave);
        best = other > best ? other : best;
    }
    if (lane_id() == 0) best_of_wave[threadIdx.x / kWave] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int v = 1; v < kArgWaves; ++v) best = best_of_wave[v] > best ? best_of_wave[v] : best;
        if (lo < hi) atomicMax(reinterpret_cast<unsigned long long *>(w.hist_a + row * kHistBins), best);
    }
}

template <bool DIFF, int UPDATE>
__global__ __launch_bounds__(kArgThreads) void argmax_finish_kernel(TopkArgs p, Ws w) {
    const int64_t row = (int64_t)blockIdx.x * kArgThreads + threadIdx.x;
    if (row >= p.n) return;
    unsigned long long *slot = reinterpret_cast<unsigned long long *>(w.hist_a + row * kHistBins);
    const int64_t e = (int64_t)(0xffffffffu - (uint32_t)(*slot & 0xffffffffull));
    *slot = 0ull;
    const float bv = DIFF ? p.b[row * p.d + e] : 0.f;
    const float v = DIFF ? p.a[row * p.d + e] - bv : p.a[row * p.d + e];
    p.out_idx[row] = (int32_t)e;                                // k == 1: one pair per row
    p.out_val[row] = v;
    if (UPDATE == kAddUpdate) p.g_i[row * p.d + e] = bv + v;    // Algorithm 2, line 6
    if (UPDATE == kClearUpdate) p.g_i[row * p.d + e] = 0.f;     // Algorithm 4
}

hipError_t launch_argmax(const TopkArgs &p, const Ws &w, hipStream_t stream, const Marker &mk) {
    const bool diff = p.b != nullptr, upd = p.g_i != nullptr;
    int64_t G = 1024 / p.n;                                     // about four workgroups of 256 per compute unit
    if (G < 1) G = 1;
    int64_t piece = (p.d + G - 1) / G;
    piece = (piece + 3) & ~(int64_t)3;
    if (piece < 4096) piece = 4096;
    G = (p.d + piece - 1) / piece;
    const dim3 grid((unsigned)G, (unsigned)p.n), block(kArgThreads);
    if (diff) hipLaunchKernelGGL(argmax_stream_kernel<true>, grid, block, 0, stream, p, w, piece);
    else hipLaunchKernelGGL(argmax_stream_kernel<false>, grid, block, 0, stream, p, w, piece);
    mk(K_TOPK_COLLECT);
    const dim3 fgrid((unsigned)((p.n + kArgThreads - 1) / kArgThreads));
    if (upd && diff) hipLaunchKernelGGL((argmax_finish_kernel<true, kAddUpdate>), fgrid, block, 0, stream, p, w);
    else if (upd) hipLaunchKernelGGL((argmax_finish_kernel<false, kClearUpdate>), fgrid, block, 0, stream, p, w);
    else if (diff) hipLaunchKernelGGL((argmax_finish_kernel<true, kNoUpdate>), fgrid, block, 0, stream, p, w);
    else hipLaunchKernelGGL((argmax_finish_kernel<false, kNoUpdate>), fgrid, block, 0, stream, p, w);
    mk(K_TOPK_SELECT);
    return hipGetLastError();
}

}  // namespace

size_t topk_split_workspace_bytes(int32_t n, int64_t d, int64_t) { return layout(n, d, nullptr, nullptr); }

hipError_t launch_topk_split_reset(void *workspace, int32_t n, int64_t d, hipStream_t stream) {
    Ws w;
    layout(n, d, (char *)workspace, &w);
    // the histograms and the row records are the leading, contiguous part of the layout
    const size_t words = ((char *)w.slot_cnt - (char *)workspace) / sizeof(uint32_t);
    size_t blocks = (words + kCandThreads - 1) / kCandThreads;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)blocks), dim3(kCandThreads), 0, stream, (uint32_t *)workspace,
                       words);
    return hipGetLastError();
}

namespace {
dim3 cand_grid(int32_t n, const Ws &w, unsigned selections) {
    return dim3((unsigned)((w.nslot + kCandWaves - 1) / kCandWaves), (unsigned)n, selections);
}

// The message index asked for, if any: a slot has to be a whole number of its blocks (see Emitter).
bool index_fits(const TopkArgs &p, const Ws &w) {
    return !p.agg_start || (p.agg_shift >= 0 && p.agg_shift < 31 && w.L % ((int64_t)1 << p.agg_shift) == 0 &&
                            p.agg_nblk == ((p.d - 1) >> p.agg_shift) + 1);
}

// Steps loaded ahead, from the candidates to be expected in a slot (1.3 k per row after a warm start, some 1.6 k from a
// sample): enough for all of them where that is few, and no more, since every wavefront loads them; `most` is what the
// kernel is compiled for.  Where a slot holds several times as many, the first load counts for less and the longer one
// only delays it.  Measured, us: ef21_topk n = 20, d = 10^6, k = 5000 (expects 68): 31.7 with two, 31.8 three, 32.4 four, 33.8
// six; step n = 8, d = 11.2 million, k = 60000 (157) 203, 202 and 198 with three, four and six; k = 92000 (240) 218, 217, 216;
// Student-t 212, 210, 208; k = 138000 (361) 234, 233, 232 and 230, 229, 224; k = 160000 (419) 236, 235, 234; k = 200000 (524)
// 250 with four, 250 with six; k = 300000 (785) 287 and 289, 280 and 283.
int cand_steps(const TopkArgs &p, const Ws &w, int most) {
    const double expected = (p.warm > 0 ? 1.3 : 1.6) * (double)p.k * (double)w.L / (double)p.d;
    int steps = 4;
    if (expected <= 90.0) steps = 2;
    else if (expected <= 150.0) steps = 3;
    else if (expected <= 450.0) steps = 6;
    return steps < most ? steps : most;
}

// After the collect pass: count (or, for a row whose warm start failed, collect again) and emit.
hipError_t launch_after_collect(const TopkArgs &p, const Ws &w, hipStream_t stream, const Marker &mk) {
    const bool diff = p.b != nullptr, upd = p.g_i != nullptr;
    const int steps = cand_steps(p, w, 6);
    const dim3 cgrid = cand_grid(p.n, w, 1), block(kCandThreads);
#define EF21_CAND(KERNEL, GRID, DIFF, UPD)                                                               \
    do {                                                                                                 \
        if (steps == 2) hipLaunchKernelGGL((KERNEL<DIFF, UPD, 2>), GRID, block, 0, stream, p, w);        \
        else if (steps == 3) hipLaunchKernelGGL((KERNEL<DIFF, UPD, 3>), GRID, block, 0, stream, p, w);   \
        else if (steps == 4) hipLaunchKernelGGL((KERNEL<DIFF, UPD, 4>), GRID, block, 0, stream, p, w);   \
        else hipLaunchKernelGGL((KERNEL<DIFF, UPD, 6>), GRID, block, 0, stream, p, w);                   \
    } while (0)
    if (upd && diff) EF21_CAND(cand_count_kernel, cgrid, true, kAddUpdate);
    else if (upd) EF21_CAND(cand_count_kernel, cgrid, false, kClearUpdate);
    else if (diff) EF21_CAND(cand_count_kernel, cgrid, true, kNoUpdate);
    else EF21_CAND(cand_count_kernel, cgrid, false, kNoUpdate);
    mk(K_TOPK_COUNT);
    if (upd && diff) EF21_CAND(cand_emit_kernel, cgrid, true, kAddUpdate);
    else if (upd) EF21_CAND(cand_emit_kernel, cgrid, false, kClearUpdate);
    else if (diff) EF21_CAND(cand_emit_kernel, cgrid, true, kNoUpdate);
    else EF21_CAND(cand_emit_kernel, cgrid, false, kNoUpdate);
#undef EF21_CAND
    mk(K_TOPK_EMIT);
    return hipGetLastError();
}
}  // namespace

// Rows of up to this size in all are found in the 256 MB of the last cache by the next round.  A round of EF, us, stored to stay
// there and streamed past: n = 8, d = 4 million (128 MB) 108 and 119; 6 million (192) 156 and 179; 7 million (224) 207 and
// 205; 9 million (288) 304 and 264.
constexpr int64_t kKeptBytes = (int64_t)200 << 20;

hipError_t launch_topk_split(const TopkArgs &p, void *workspace, hipStream_t stream, const Marker &mk) {
    Ws w;
    layout(p.n, p.d, (char *)workspace, &w);
    w.rule = sample_rule(p.k, p.d);
    if (p.g_i && p.g_i != (p.b ? p.b : p.a)) return hipErrorInvalidValue;
    if (p.warm < 0 || p.warm > kWarmSlots) return hipErrorInvalidValue;
    if (!index_fits(p, w) || (p.agg_start && p.k == 1)) return hipErrorInvalidValue;
    if (p.add && (p.b || p.g_i != p.a || p.warm == 0 || p.k == 1)) return hipErrorInvalidValue;
    if (p.k == 1) return launch_argmax(p, w, stream, mk);
    const dim3 add_grid((unsigned)w.G, (unsigned)p.n), block(kBlk);
    if (p.add && (int64_t)p.n * p.d * 4 <= kKeptBytes)
        hipLaunchKernelGGL((split_collect_kernel<false, kWarmPass, kAddKept>), add_grid, block, 0, stream, p, w);
    else if (p.add)
        hipLaunchKernelGGL((split_collect_kernel<false, kWarmPass, kAddStreamed>), add_grid, block, 0, stream, p, w);
    else
        launch_collect(p, w, stream);
    mk(K_TOPK_COLLECT);
    hipError_t st = hipGetLastError();
    if (st != hipSuccess) return st;
    return launch_after_collect(p, w, stream, mk);
}

int64_t topk_split_slots(int32_t n, int64_t d) {
    Ws w;
    plan(n, d, &w);
    return w.nslot;
}

int64_t topk_split_slot_entries(int32_t n, int64_t d) {
    Ws w;
    plan(n, d, &w);
    return w.nslot * w.L;
}

hipError_t launch_topk_split_pair(const TopkArgs &plain, const TopkArgs &markov, void *ws_plain, void *ws_markov,
                                  const PairSums &sums, hipStream_t stream, const Marker &mk) {
    if (plain.b || !markov.b || plain.a != markov.a || plain.n != markov.n || plain.d != markov.d ||
        plain.k != markov.k || plain.g_i || markov.g_i || plain.k < 2 || plain.warm < 0 || plain.warm > kWarmSlots ||
        markov.warm < 0 || markov.warm > kWarmSlots || (plain.warm > 0) != (markov.warm > 0) || !sums.norms ||
        !sums.kept_plain || !sums.kept_markov)
        return hipErrorInvalidValue;
    Ws wp, wm;
    layout(plain.n, plain.d, (char *)ws_plain, &wp);
    layout(markov.n, markov.d, (char *)ws_markov, &wm);
    if (!index_fits(plain, wp) || !index_fits(markov, wm)) return hipErrorInvalidValue;
    wp.rule = wm.rule = sample_rule(plain.k, plain.d);
    wp.kept = sums.kept_plain;
    wm.kept = sums.kept_markov;
    wm.resid = sums.resid;
    const bool warm = markov.warm > 0;
    const dim3 grid((unsigned)wm.G, (unsigned)markov.n), block(kBlk);
    double2 *norms = (double2 *)sums.norms;
    if (warm) hipLaunchKernelGGL(split_collect_pair_kernel<true>, grid, block, 0, stream, markov, wm, plain.warm, wp, norms);
    else hipLaunchKernelGGL(split_collect_pair_kernel<false>, grid, block, 0, stream, markov, wm, plain.warm, wp, norms);
    mk(K_TOPK_COLLECT);
    const int steps = cand_steps(markov, wm, 4);
    const dim3 cgrid = cand_grid(markov.n, wm, 2);
#define EF21_CAND(KERNEL)                                                                                \
    do {                                                                                                 \
        if (steps == 2) hipLaunchKernelGGL(KERNEL<2>, cgrid, block, 0, stream, plain, wp, markov, wm);   \
        else if (steps == 3) hipLaunchKernelGGL(KERNEL<3>, cgrid, block, 0, stream, plain, wp, markov, wm); \
        else hipLaunchKernelGGL(KERNEL<4>, cgrid, block, 0, stream, plain, wp, markov, wm);              \
    } while (0)
    EF21_CAND(cand_count_pair_kernel);
    mk(K_TOPK_COUNT);
    EF21_CAND(cand_emit_pair_kernel);
#undef EF21_CAND
    mk(K_TOPK_EMIT);
    return hipGetLastError();
}

}  // namespace ef21
