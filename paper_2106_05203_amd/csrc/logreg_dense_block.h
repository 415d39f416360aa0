// The one-pass dense gradient of eq. (9) as device code shared by the kernels that run it (the gradient kernel
// and the fused small-problem iteration), so that both produce the same bits: the plan that cuts a worker's
// rows into blocks, and the work of one block of kDenseWaves wavefronts.
#pragma once
#include <type_traits>
#include <utility>

#include "device_utils.h"
#include "logreg_finish.h"

namespace ef21 {

constexpr int kDenseThreads = 256;                    // threads of one row block
constexpr int kDenseWaves = kDenseThreads / kWave;

struct DensePlan {
    int64_t rows_per_wg;
    int64_t chunks;   // row blocks per worker
};

// Row blocks per worker that the partial sums have room for: about two workgroups per compute unit over all workers.
inline int64_t max_chunks(int32_t n, int64_t m) {
    const int64_t target = (512 + n - 1) / n, by_rows = (m + 3) / 4;
    return by_rows < target ? by_rows : target;
}

// Row `l` of a worker's batch: the row of A it names, or -1 when the entry lies outside [0, m_full) (such an
// entry contributes nothing and is never dereferenced).
__device__ __forceinline__ int64_t batch_row(const int32_t *__restrict__ batch, int64_t at, int64_t m_full) {
    const uint32_t b = (uint32_t)batch[at];
    return b < (uint64_t)m_full ? (int64_t)b : -1;
}

// Which instantiation of dense_block serves rows of d columns (the kernels that must agree bit for bit choose through
// this one function): LANES lanes of a wavefront per row, NQ quads of columns per lane.  {0, 0}: none (a workgroup per
// row, or two passes).  Rows longer than 2048 whose length is no multiple of four go to the workgroup-per-row kernel.
struct DenseVariant {
    int lanes, nq;
};
enum RowShape { kQuadRows = 0 /* d % 4 == 0 */, kRaggedRows = 1, kTinyRows = 2 /* d < 4 */ };

inline DenseVariant dense_variant(int64_t d) {
    if (d <= 64) return {16, 1};
    if (d <= 128) return {32, 1};
    if (d <= 256) return {64, 1};
    if (d <= 512) return {64, 2};
    if (d <= 1024) return {64, 4};
    if (d <= 2048) return {64, 8};
    if (d <= 4096 && d % 4 == 0) return {64, 16};
    return {0, 0};
}

// Rows in flight per group of LANES lanes: 32 row entries per lane for short rows of small problems (more does not fit
// the registers of the 1024-thread kernel that shares this code), 64 otherwise (`deep`: n = 16, m = 8000, d = 60, 31 MB, the whole
// gradient 11.6 us with 32 entries, 10.9 with 64); one row where a row alone fills the registers.
constexpr int64_t kSmallProblem = (int64_t)1 << 24;                       // n * m * d
template <int LANES, int NQ, bool DEEP>
constexpr int dense_rows_in_flight() {
    if (NQ >= 8) return NQ == 8 ? 2 : 1;
    return (LANES == 16 ? 4 : 8 / NQ) * (DEEP ? 2 : 1);
}
inline bool dense_deep(int32_t n, int64_t m_full, int64_t d) { return (int64_t)n * m_full * d > kSmallProblem; }

// Rows that a block of kDenseWaves wavefronts takes per trip, for rows of d columns.
inline int64_t dense_trip_rows(int64_t d, bool deep) {
    const DenseVariant v = dense_variant(d);
    if (v.nq >= 8) return kDenseWaves * (v.nq == 8 ? 2 : 1);
    return (v.lanes == 64 ? kDenseWaves * (8 / v.nq) : 64) * (deep ? 2 : 1);
}

// About two workgroups per compute unit in all (512 on 256 CUs), each streaming one long block of rows:
// fewer, longer blocks measured faster than several rounds of short ones, and they leave fewer partial
// sums to add.  At least 8 rows each, 32 short ones (12 KB): below that the sums cost more than the rows.  One block
// more where that saves every block a trip.
inline DensePlan dense_plan(int32_t n, int64_t m, int64_t d, bool deep) {
    int64_t target = 512 / n;
    if (target < 1) target = 1;
    const int64_t trip = dense_trip_rows(d, deep), least = d <= 128 ? 32 : (d <= 256 ? 16 : 8);
    int64_t rows = (m + target - 1) / target;
    const int64_t fewer = (m + max_chunks(n, m) - 1) / max_chunks(n, m);
    if ((fewer + trip - 1) / trip < (rows + trip - 1) / trip) rows = fewer;
    // Small problems: half as many blocks, one per compute unit, of about 100 KB of rows or more, but 32 per worker in any
    // case: each block's sums are read again.  The gradient of n = 1, m = 8000, d = 1000: 34 us with 500 blocks, 31 with 32,
    // 16.3 so; n = 1, m = 100000, d = 80: 42, 95, 23; n = 8, m = 1000, d = 1000: 14.4, 11.1, 11.1.  step of n = 5, m = 700,
    // d = 1001: 17.9 us with 32 blocks per worker, 19.2 with 42.  Above 2^23 entries: m = 20000, d = 1000 30 us with 512 blocks
    // and 25 with 256, but m = 200000, d = 80 31 and 35, n = 8, m = 8000, d = 300 19.6 and 25.9.
    if ((int64_t)n * m * d <= ((int64_t)1 << 23)) {
        int64_t most = m * d / 24576 < 256 / n ? m * d / 24576 : 256 / n;
        if (most < 48) most = 32;                              // (a few more gain nothing)
        if (rows < (m + most - 1) / most) rows = (m + most - 1) / most;
    }
    if (rows < least) rows = least;
    return {rows, (m + rows - 1) / rows};
}

// Entry r of v, r < ROWS a power of two.
template <int ROWS, class T>
__device__ __forceinline__ T pick_row(const T (&v)[ROWS], int r) {
    static_assert((ROWS & (ROWS - 1)) == 0, "halves");
    T t[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) t[i] = v[i];
#pragma unroll
    for (int w = ROWS / 2; w > 0; w /= 2)
#pragma unroll
        for (int i = 0; i < w; ++i) t[i] = (r & w) ? t[i + w] : t[i];
    return t[0];
}

// Which of ROWS rows (a power of two up to 16) a lane stands for in fold_rows and spread_rows, and a lane of each row of
// sixteen lanes that stands for row r.  Bits 0 and 1 are turned in every other four lanes and bit 2 in the upper eight, so that the
// lanes that mirror one another (DPP row_half_mirror, row_mirror) stand for the same row until their turn to divide rows.
template <int ROWS>
__device__ __forceinline__ int row_of_lane() {
    const int i = lane_id(), b2 = (i >> 2) & 1, b3 = (i >> 3) & 1;
    return (((i & 3) ^ (b2 ? 3 : 0)) | ((b2 ^ b3) << 2) | (b3 << 3)) & (ROWS - 1);
}
constexpr int lane_of_row(int r) {
    const int b3 = (r >> 3) & 1, b2 = ((r >> 2) & 1) ^ b3;
    return ((r & 3) ^ (b2 ? 3 : 0)) | (b2 << 2) | (b3 << 3);
}

// Sums of v[0..ROWS) over each group of LANES lanes, the same bits as group_sum: lane i receives that of row
// row_of_lane().  At each of the first steps the two lanes of a pair divide their rows between them and exchange the halves,
// so ROWS sums take little more than one: 30 instructions for eight rows where eight group_sums take 160.
template <int LANES, int ROWS>
__device__ __forceinline__ float fold_rows(const float (&v)[ROWS]) {
    const int mine = row_of_lane<16>();
    float t[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) t[i] = v[i];
    // rows that differ in the lowest bit lie side by side: the kept one, plus what the partner sends of it
    auto halve = [&](auto ctrl, auto count, int bit) {
        constexpr int kCtrl = decltype(ctrl)::value, kCount = decltype(count)::value;
        if constexpr (kCount > 1) {
            const bool upper = (mine >> bit) & 1;
#pragma unroll
            for (int i = 0; i < kCount / 2; ++i) {
                const float keep = upper ? t[2 * i + 1] : t[2 * i], send = upper ? t[2 * i] : t[2 * i + 1];
                t[i] = keep + dpp_move<kCtrl>(send);
            }
        } else {
            t[0] += dpp_move<kCtrl>(t[0]);
        }
    };
    halve(std::integral_constant<int, 0xB1>(), std::integral_constant<int, ROWS>(), 0);           // quad_perm [1,0,3,2]
    halve(std::integral_constant<int, 0x4E>(), std::integral_constant<int, (ROWS + 1) / 2>(), 1); // quad_perm [2,3,0,1]
    halve(std::integral_constant<int, 0x141>(), std::integral_constant<int, (ROWS + 3) / 4>(), 2); // row_half_mirror
    halve(std::integral_constant<int, 0x140>(), std::integral_constant<int, (ROWS + 7) / 8>(), 3); // row_mirror
    float s = t[0];
    if constexpr (LANES >= 32) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(s), false, false);
        s = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    if constexpr (LANES == 64) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
        s = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    return s;
}

// v[r] = the value of the lane of the caller's row of sixteen lanes that stands for row r (DPP row_newbcast).
template <int ROWS, int... R>
__device__ __forceinline__ void spread_rows_impl(float own, float (&v)[ROWS], std::integer_sequence<int, R...>) {
    ((v[R] = dpp_move<0x150 + lane_of_row(R)>(own)), ...);
}
template <int ROWS>
__device__ __forceinline__ void spread_rows(float own, float (&v)[ROWS]) {
    static_assert(ROWS <= 16, "lanes of a row");
    spread_rows_impl(own, v, std::make_integer_sequence<int, ROWS>());
}

// The rows [l0, l1) of `worker`, shared by `waves` wavefronts (`wave` = the caller's number among them): this lane's part of
// sum_l coef_l a_l, added to acc.  A group of LANES lanes owns whole
// rows; a lane keeps its columns of the row, NQ quads, in registers between the dot product (a sum over the group) and
// the rank-one accumulation coef * a_l.  Rows need no alignment: in ragged rows (d no multiple of four) the quad that
// straddles the end of the row is moved back onto its last four columns, those of them that belong to the quad before
// it count as zero; rows of less than four columns are read one by one.
// Where rows are short the sums over a group, the exponential and the division of a row cost more than its products, so the rows of
// a trip are summed together and every lane works out the coefficient of one of them (fold_rows, spread_rows): the gradient of
// n = 1, m = 200000, d = 80 31.6 -> 26.0 us, 2, 40000, 250 29.1 -> 22.6, 32, 8000, 60 16.3 -> 13.9, the same bits.
// BATCH: the m rows of a worker are the entries of batch[worker][0..m) (row numbers inside its m_full rows), the
// minibatch of Algorithm 5, read one trip ahead; otherwise m_full == m and row l is row l.
// n = 20, m = 1628, d = 123 (16 MB): 10.5 us with four-byte loads and a wavefront per row, 6.7 so; a minibatch of 625 of
// 5000 rows of 2000 (100 MB): 25.1 -> 21.3 us.
template <int LANES, int NQ, int ROWS, int SHAPE, bool BATCH, int WAVES, class Acc>
__device__ __forceinline__ void dense_rows(const float *__restrict__ A, const float *__restrict__ y,
                                           const float *__restrict__ x, int64_t m, int64_t d, int64_t l0, int64_t l1,
                                           int loss, const int32_t *__restrict__ batch, int64_t m_full, int64_t worker,
                                           int wave, Acc (&acc)[NQ][4]) {
    constexpr int kGroups = kWave / LANES;    // rows side by side
    constexpr bool kKept = std::is_same_v<Acc, double>;       // few rows, which the next call finds in L2
    const int lane = lane_id(), sub = lane % LANES, group = lane / LANES;

    int32_t at[NQ];                           // where the quad is read
    int dup[NQ];                              // its leading columns that are another quad's; 4: past the end of the row
    float xr[NQ][4];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int32_t c0 = (q * LANES + sub) * 4, last = (int32_t)d - 4;
        at[q] = SHAPE == kTinyRows ? 0 : (c0 < last ? c0 : last);
        dup[q] = c0 - at[q] < 4 ? c0 - at[q] : 4;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float xv = SHAPE != kTinyRows || t < d ? x[at[q] + t] : 0.f;
            xr[q][t] = t >= dup[q] ? xv : 0.f;
            acc[q][t] = (Acc)0;
        }
    }

    // ROWS rows per group and trip: their loads are all issued before the first dot product.  A row index past the
    // block is clamped to the block's last row, an entry of the batch that names no row to row 0; what they load is
    // cleared and their coefficient set to zero (an infinity times that zero would be NaN).
    constexpr int64_t kTrip = (int64_t)WAVES * ROWS * kGroups;
    auto listed = [&](int64_t l, int32_t (&src)[ROWS]) {          // row numbers of a trip
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int64_t lr = l + r * kGroups + group < l1 ? l + r * kGroups + group : l1 - 1;
            src[r] = (int32_t)(BATCH ? batch_row(batch, worker * m + lr, m_full) : lr);
        }
    };
    const int mine = row_of_lane<ROWS>();
    int32_t src[ROWS];
    const int64_t first = l0 + wave * ROWS * kGroups;
    if (first < l1) listed(first, src);
    for (int64_t l = first; l < l1; l += kTrip) {
        float av[ROWS][NQ][4], s[ROWS];
        bool live[ROWS];
        // the row whose coefficient this lane works out
        const int64_t mine_l = l + mine * kGroups + group;
        const int32_t mine_src = BATCH ? pick_row(src, mine) : (int32_t)(mine_l < l1 ? mine_l : l1 - 1);
        const bool mine_live = mine_l < l1 && mine_src >= 0;
        const float mine_y = y[worker * m_full + (mine_src > 0 ? mine_src : 0)];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            live[r] = l + r * kGroups + group < l1 && (!BATCH || src[r] >= 0);
            const int64_t lr = BATCH && src[r] < 0 ? 0 : (int64_t)src[r];
            const float *row = A + (worker * m_full + lr) * d;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                if constexpr (SHAPE == kTinyRows) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) av[r][q][t] = t < d ? stream_load(row + t) : 0.f;
                } else {
                    const float4 t4 = kKept ? load4_any(row + at[q]) : stream_load4_any(row + at[q]);
                    av[r][q][0] = SHAPE == kRaggedRows && dup[q] > 0 ? 0.f : t4.x;
                    av[r][q][1] = SHAPE == kRaggedRows && dup[q] > 1 ? 0.f : t4.y;
                    av[r][q][2] = SHAPE == kRaggedRows && dup[q] > 2 ? 0.f : t4.z;
                    av[r][q][3] = t4.w;
                }
            }
        }
        if (l + kTrip < l1) listed(l + kTrip, src);
        bool clear = l + ROWS * kGroups > l1;                     // a block's last trip
        if constexpr (BATCH) {
            bool named = true;
#pragma unroll
            for (int r = 0; r < ROWS; ++r) named = named && live[r];
            clear = !__all(named);
        }
        if (clear) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
#pragma unroll
                for (int q = 0; q < NQ; ++q)
#pragma unroll
                    for (int t = 0; t < 4; ++t) av[r][q][t] = live[r] ? av[r][q][t] : 0.f;
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            s[r] = 0.f;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                float p = s[r];
#pragma unroll
                for (int t = 0; t < 4; ++t) p = fmaf(av[r][q][t], xr[q][t], p);
                s[r] = dup[q] < 4 ? p : s[r];                     // (an infinity of another column times zero)
            }
        }
        const float margin = fold_rows<LANES>(s), own_coef = mine_live ? loss_derivative(mine_y, margin, loss) : 0.f;
        float coef[ROWS];
        spread_rows(own_coef, coef);
        if constexpr (std::is_same_v<Acc, double>) {
            // Two rows in fp32, then to the sum: the roundings stay below those of the separate kernels, which add eight
            // rows and more before fp64 takes over.
            static_assert(ROWS % 2 == 0, "pairs");
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int r = 0; r < ROWS; r += 2)
                        acc[q][t] += (double)fmaf(coef[r + 1], av[r + 1][q][t], coef[r] * av[r][q][t]);
        } else {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
#pragma unroll
                for (int q = 0; q < NQ; ++q)
#pragma unroll
                    for (int t = 0; t < 4; ++t) acc[q][t] = fmaf(coef[r], av[r][q][t], acc[q][t]);
            }
        }
    }
}

// One row block: rows [chunk * rows_per_wg, +rows_per_wg) of `worker`, by kDenseWaves wavefronts (`wave` = this
// wavefront's number among them, `tid` = the thread's among their kDenseThreads), see dense_rows.
// `red` (NQ * LANES * 4 floats of LDS, the block's own) adds the wavefronts' accumulators in
// wavefront order; the result goes to part[worker][chunk][0..d).  Every thread of the workgroup must call (it holds
// workgroup barriers); `active` = false does no work and writes nothing.
template <int LANES, int NQ, int ROWS, int SHAPE, bool BATCH>
__device__ __forceinline__ void dense_block(const float *__restrict__ A, const float *__restrict__ y,
                                            const float *__restrict__ x, float *__restrict__ part, int64_t m,
                                            int64_t d, int64_t rows_per_wg, int loss,
                                            const int32_t *__restrict__ batch, int64_t m_full, int64_t worker,
                                            int64_t chunk, int64_t chunks, int wave, int tid, bool active,
                                            float *red) {
    constexpr int kCols = NQ * LANES * 4;     // columns covered by one group
    const int lane = lane_id(), sub = lane % LANES, group = lane / LANES;
    const int64_t l0 = chunk * rows_per_wg;
    const int64_t l1 = !active ? l0 : (l0 + rows_per_wg < m ? l0 + rows_per_wg : m);
    float acc[NQ][4];
    dense_rows<LANES, NQ, ROWS, SHAPE, BATCH, kDenseWaves>(A, y, x, m, d, l0, l1, loss, batch, m_full, worker, wave, acc);

    // the groups of a wavefront, then the wavefronts in order
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int o = LANES; o < kWave; o <<= 1) acc[q][t] += __shfl_xor(acc[q][t], o, kWave);
    for (int w = 0; w < kDenseWaves; ++w) {
        if (wave == w && group == 0) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                float4 *slot = reinterpret_cast<float4 *>(red) + q * LANES + sub;
                float4 sum = make_float4(acc[q][0], acc[q][1], acc[q][2], acc[q][3]);
                if (w > 0) {
                    const float4 before = *slot;
                    sum = make_float4(before.x + sum.x, before.y + sum.y, before.z + sum.z, before.w + sum.w);
                }
                *slot = sum;
            }
        }
        __syncthreads();
    }
    // entry e of `red` is entry e % 4 of quad e / 4, which was read at min(e / 4 * 4, d - 4): the straddling quad's
    // leading columns are another's
    if (active) {
        float *out = part + (worker * chunks + chunk) * d;
        for (int e = tid; e < kCols; e += kDenseThreads) {
            const int32_t c0 = e & ~3, last = SHAPE == kTinyRows ? 0 : (int32_t)d - 4, c = (c0 < last ? c0 : last) + (e & 3);
            if (c >= c0 && c < d) out[c] = red[e];
        }
    }
}

// The whole gradient of one worker by one workgroup of kSoloWaves wavefronts, without partial sums in memory: the lanes'
// sums and the wavefronts' are in fp64, the latter added in LDS (`lds`: kSoloWaves * NQ * LANES * 4 doubles) in a fixed
// order.  put(c, entry) is called for every column c < d by thread c; every thread of the workgroup must call, and a barrier
// has to follow before `lds` is used again.
constexpr int kSoloThreads = 1024, kSoloWaves = kSoloThreads / kWave;
template <int LANES, int NQ, int SHAPE, bool BATCH, class PutFn>
__device__ __forceinline__ void solo_gradient(const float *__restrict__ A, const float *__restrict__ y,
                                              const float *__restrict__ x, int64_t m, int64_t d, float lambda, int loss,
                                              const int32_t *__restrict__ batch, int64_t m_full, int64_t worker,
                                              double *lds, PutFn put) {
    constexpr int kCols = NQ * LANES * 4;
    static_assert(kCols <= kSoloThreads, "a column per thread");
    const int tid = threadIdx.x, wave = wave_id(), lane = lane_id(), sub = lane % LANES;
    const float x_c = tid < d ? x[tid] : 0.f;
    double acc[NQ][4];
    dense_rows<LANES, NQ, dense_rows_in_flight<LANES, NQ, false>(), SHAPE, BATCH, kSoloWaves>(A, y, x, m, d, 0, m, loss, batch,
                                                                                           m_full, worker, wave, acc);
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
#pragma unroll
            for (int o = LANES; o < kWave; o <<= 1) acc[q][t] += __shfl_xor(acc[q][t], o, kWave);
            if (lane < LANES) lds[wave * kCols + (q * LANES + sub) * 4 + t] = acc[q][t];
        }
    __syncthreads();
    if (tid < d) {
        // column c is entry c % 4 of quad c / 4; the quad that straddles the end of the row was read at d - 4
        const int c0 = tid & ~3, last = SHAPE == kTinyRows ? 0 : (int)d - 4, e = c0 < last ? tid : c0 + tid - last;
        double s[4] = {};
#pragma unroll
        for (int w = 0; w < kSoloWaves; ++w) s[w % 4] += lds[w * kCols + (SHAPE == kTinyRows ? tid : e)];
        put(tid, dense_grad_of_sum((s[0] + s[1]) + (s[2] + s[3]), x_c, m, lambda));
    }
}

}  // namespace ef21
