// The one-pass dense gradient of eq. (9) as device code shared by the kernels that run it (the gradient kernel
// and the fused small-problem iteration), so that both produce the same bits: the plan that cuts a worker's
// rows into blocks, and the work of one block of kDenseWaves wavefronts.
#pragma once
#include "device_utils.h"

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

// One row block: rows [chunk * rows_per_wg, +rows_per_wg) of `worker`, by kDenseWaves wavefronts (`wave` = this
// wavefront's number among them, `tid` = the thread's among their kDenseThreads).  A group of LANES lanes owns whole
// rows; a lane keeps its columns of the row, NQ quads, in registers between the dot product (a sum over the group) and
// the rank-one accumulation coef * a_l.  Rows need no alignment: in ragged rows (d no multiple of four) the quad that
// straddles the end of the row is moved back onto its last four columns, those of them that belong to the quad before
// it count as zero; rows of less than four columns are read one by one.  `red` (NQ * LANES * 4 floats of LDS, the block's own) adds the wavefronts' accumulators in
// wavefront order; the result goes to part[worker][chunk][0..d).  Every thread of the workgroup must call (it holds
// workgroup barriers); `active` = false does no work and writes nothing.
// BATCH: the m rows of a worker are the entries of batch[worker][0..m) (row numbers inside its m_full rows), the
// minibatch of Algorithm 5, read one trip ahead; otherwise m_full == m and row l is row l.
// n = 20, m = 1628, d = 123 (16 MB): 10.5 us with four-byte loads and a wavefront per row, 6.7 so; a minibatch of 625 of
// 5000 rows of 2000 (100 MB): 25.1 -> 21.3 us.
template <int LANES, int NQ, int ROWS, int SHAPE, bool BATCH>
__device__ __forceinline__ void dense_block(const float *__restrict__ A, const float *__restrict__ y,
                                            const float *__restrict__ x, float *__restrict__ part, int64_t m,
                                            int64_t d, int64_t rows_per_wg, int loss,
                                            const int32_t *__restrict__ batch, int64_t m_full, int64_t worker,
                                            int64_t chunk, int64_t chunks, int wave, int tid, bool active,
                                            float *red) {
    constexpr int kCols = NQ * LANES * 4;     // columns covered by one group
    constexpr int kGroups = kWave / LANES;    // rows side by side
    const int lane = lane_id(), sub = lane % LANES, group = lane / LANES;

    int32_t at[NQ];                           // where the quad is read
    int dup[NQ];                              // its leading columns that are another quad's; 4: past the end of the row
    float xr[NQ][4], acc[NQ][4];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int32_t c0 = (q * LANES + sub) * 4, last = (int32_t)d - 4;
        at[q] = SHAPE == kTinyRows ? 0 : (c0 < last ? c0 : last);
        dup[q] = c0 - at[q] < 4 ? c0 - at[q] : 4;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float xv = SHAPE != kTinyRows || t < d ? x[at[q] + t] : 0.f;
            xr[q][t] = t >= dup[q] ? xv : 0.f;
            acc[q][t] = 0.f;
        }
    }

    // ROWS rows per group and trip: their loads are all issued before the first dot product.  A row index past the
    // block is clamped to the block's last row, an entry of the batch that names no row to row 0; what they load is
    // cleared and their coefficient set to zero (an infinity times that zero would be NaN).
    const int64_t l0 = chunk * rows_per_wg;
    const int64_t l1 = !active ? l0 : (l0 + rows_per_wg < m ? l0 + rows_per_wg : m);
    constexpr int64_t kTrip = (int64_t)kDenseWaves * ROWS * kGroups;
    auto listed = [&](int64_t l, int64_t (&src)[ROWS]) {          // row numbers of a trip
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int64_t lr = l + r * kGroups + group < l1 ? l + r * kGroups + group : l1 - 1;
            src[r] = BATCH ? batch_row(batch, worker * m + lr, m_full) : lr;
        }
    };
    int64_t src[ROWS];
    const int64_t first = l0 + wave * ROWS * kGroups;
    if (first < l1) listed(first, src);
    for (int64_t l = first; l < l1; l += kTrip) {
        float av[ROWS][NQ][4], yl[ROWS], s[ROWS];
        bool live[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            live[r] = l + r * kGroups + group < l1 && (!BATCH || src[r] >= 0);
            const int64_t lr = BATCH && src[r] < 0 ? 0 : src[r];
            const float *row = A + (worker * m_full + lr) * d;
            yl[r] = y[worker * m_full + lr];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                if constexpr (SHAPE == kTinyRows) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) av[r][q][t] = t < d ? stream_load(row + t) : 0.f;
                } else {
                    const float4 t4 = stream_load4_any(row + at[q]);
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
#pragma unroll
        for (int r = 0; r < ROWS; ++r) s[r] = group_sum<LANES>(s[r]);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const float coef = live[r] ? loss_derivative(yl[r], s[r], loss) : 0.f;
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[q][t] = fmaf(coef, av[r][q][t], acc[q][t]);
        }
    }

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

}  // namespace ef21
