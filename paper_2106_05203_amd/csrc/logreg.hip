// Local gradients of the objective of Section 5, eq. (9), for all workers:
//   grad f_i(x) = (1/m) sum_l  -y_l / (1 + exp(y_l a_l^T x)) a_l  +  2 lambda x_j / (1 + x_j^2)^2.
//
// These are GEMV-shaped (each matrix entry is used twice, about one flop per byte), far below
// the matrix-core ridge, so they are written as coalesced streaming kernels, not MFMA tiles.
//
// Dense rows, d <= 4096: ONE pass over A.  A group of lanes owns whole rows; a lane keeps its columns
// of the row in registers between the dot product (a sum over the group, no LDS) and the rank-one
// accumulation r_l * a_l into per-lane accumulators.  Workgroups write partial sums that a small
// second kernel adds in a fixed order (bitwise reproducible), together with the regulariser.
// Dense rows, d up to 28672: the same with a workgroup per row (logreg_dense_wide_kernel).
// Dense rows, larger d: z = A x, then A^T r, two passes.  (CSR rows: logreg_csr.hip.)
#include "device_utils.h"
#include "kernels.h"
#include "logreg_dense_block.h"
#include "logreg_finish.h"

namespace ef21 {
namespace {

constexpr int kThreads = kDenseThreads;
constexpr int kWaves = kDenseWaves;

// ------------------------------------------------------------------ dense, one pass over A
template <int LANES, int NQ, bool DEEP, int SHAPE, bool BATCH>
__global__ __launch_bounds__(kThreads) void logreg_dense_fused_kernel(const float *__restrict__ A,
                                                                      const float *__restrict__ y,
                                                                      const float *__restrict__ x,
                                                                      float *__restrict__ part, int64_t m,
                                                                      int64_t d, int64_t rows_per_wg, int loss,
                                                                      const int32_t *__restrict__ batch,
                                                                      int64_t m_full, int64_t x_stride) {
    __shared__ __attribute__((aligned(16))) float red[NQ * LANES * 4];
    const int64_t worker = blockIdx.y;
    dense_block<LANES, NQ, dense_rows_in_flight<LANES, NQ, DEEP>(), SHAPE, BATCH>(A, y, x + worker * x_stride /* 0: one x for all workers */, part, m, d,
                                      rows_per_wg, loss, batch, m_full, worker, blockIdx.x, gridDim.x,
                                      wave_id(), threadIdx.x, true, red);
}

// ------------------------------------------------------------------ dense, wide rows, one pass over A
// Rows too long for one wavefront's registers: a workgroup of 1024 threads owns whole rows, a thread NQ quads of
// columns (quad q of thread t: columns 4 (1024 q + t) ..).  The dot product is a wavefront sum, sixteen values in
// LDS and one barrier per group of R rows; the rank-one accumulation stays in registers, so A is read once.  HBM
// bandwidth bounds it: the next group's loads are issued before this group is summed (two register buffers, the
// barriers order LDS only), and one workgroup per compute unit keeps 1024 threads x R x NQ x 16 bytes in flight.
// Rows need no alignment: the quad that straddles the end of the row is moved back onto the row's last four
// columns, its columns that belong to the quad before it count as zero and are not written (RAGGED); quads past the
// end read the same place and are dropped.  From NQ = 5 on x lives in LDS instead of registers.
// The whole gradient, n = 8, m = 2000, d = 12000 (768 MB): 124 us, 6.2 TB/s, against 461 us for the two passes below;
// n = 8, m = 1200, d = 20001: 149 against 564; n = 2, m = 100, d = 4097: 10.1 against 18.0.
constexpr int kWideThreads = 1024, kWideWaves = kWideThreads / kWave;
constexpr int64_t kWideMax = 7 * 4 * kWideThreads;        // columns (with eight quads the compiler spills)

template <int NQ>
constexpr int wide_rows() {                               // rows per group
    return NQ <= 2 ? 4 : (NQ <= 4 ? 2 : 1);
}

// Chains of additions are kept short.  Where a group is one row: two chunks per workgroup, half as many rows each.
// Elsewhere x is in registers and LDS is free: every kFoldGroups groups the accumulators move to LDS (a slot per
// thread, no barrier).  Error of the gradient of n = 8, m = 2000, d = 12000 against 64 bits: 1.1e-7 without the fold.
constexpr int kFoldGroups = 8;
template <int NQ>
constexpr int wide_chunks() {
    return wide_rows<NQ>() == 1 ? 2 : 1;
}

template <int NQ, bool RAGGED, bool BATCH>
__global__ __launch_bounds__(kWideThreads) void logreg_dense_wide_kernel(const float *__restrict__ A,
                                                                         const float *__restrict__ y,
                                                                         const float *__restrict__ x,
                                                                         float *__restrict__ part, int64_t m, int64_t d,
                                                                         int64_t rows_per_chunk, int64_t chunks,
                                                                         int loss, const int32_t *__restrict__ batch,
                                                                         int64_t m_full, int64_t x_stride) {
    constexpr int R = wide_rows<NQ>();
    constexpr bool kXLds = NQ >= 5;
    __shared__ float sums[2][R][kWideWaves];
    constexpr bool kFold = R > 1;
    static_assert(!(kXLds && kFold), "x and the folded sums do not both fit LDS");
    __shared__ float4 x_lds[kXLds ? NQ * kWideThreads : 1];
    __shared__ float4 folded[kFold ? NQ * kWideThreads : 1];
    const int64_t worker = blockIdx.y;
    const int tid = threadIdx.x, wave = tid / kWave, lane = lane_id();
    const float *xw = x + worker * x_stride;
    const int32_t last = (int32_t)d - 4;

    int32_t at[NQ];                // where the quad is read
    int dup[NQ];                   // its leading columns that are another quad's; 4: past the end of the row
    float xr[kXLds ? 1 : NQ][4], acc[NQ][4];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int32_t c0 = (q * kWideThreads + tid) * 4;
        at[q] = c0 < last ? c0 : last;
        dup[q] = c0 - at[q] < 4 ? c0 - at[q] : 4;
        float xq[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            xq[t] = t >= dup[q] ? xw[at[q] + t] : 0.f;
            acc[q][t] = 0.f;
            if constexpr (!kXLds) xr[q][t] = xq[t];
        }
        if constexpr (kXLds) x_lds[q * kWideThreads + tid] = make_float4(xq[0], xq[1], xq[2], xq[3]);   // own use only
        if constexpr (kFold) folded[q * kWideThreads + tid] = make_float4(0.f, 0.f, 0.f, 0.f);
    }

    // the block's chunks of rows; each leaves its own partial sums
    constexpr int64_t kChunks = wide_chunks<NQ>();
    int64_t chunk = (int64_t)blockIdx.x * kChunks;
    const int64_t l0 = chunk * rows_per_chunk;
    const int64_t l1 = l0 + kChunks * rows_per_chunk < m ? l0 + kChunks * rows_per_chunk : m;
    // the loads of rows l .. l + R - 1; a row past the block, or an entry of the batch that names no row, reads the first
    // 16 bytes of A (one cached line) and is cleared before it is used
    auto load = [&](int64_t l, float4 (&v)[R][NQ], float (&yl)[R], bool (&live)[R]) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            live[r] = l + r < l1;
            int64_t src = live[r] ? l + r : l0;
            if constexpr (BATCH) {
                src = batch_row(batch, worker * m + src, m_full);
                if (src < 0) {
                    src = 0;
                    live[r] = false;
                }
            }
            const float *row = live[r] ? A + (worker * m_full + src) * d : A;
            yl[r] = y[worker * m_full + src];
#pragma unroll
            for (int q = 0; q < NQ; ++q) v[r][q] = stream_load4_any(row + (live[r] ? at[q] : 0));
        }
    };
    float4 av[R][NQ], next[R][NQ];
    float yl[R], y_next[R];
    bool live[R], live_next[R];
    load(l0, av, yl, live);
    int buf = 0, unfolded = 0;
    for (int64_t l = l0; l < l1; l += R, buf ^= 1) {
        load(l + R, next, y_next, live_next);
        if (BATCH || l + R > l1) {                             // (an infinity there times a zero coefficient would be NaN)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (live[r]) continue;                         // uniform
#pragma unroll
                for (int q = 0; q < NQ; ++q) av[r][q] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float s = 0.f;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                float4 xq;
                if constexpr (kXLds) xq = x_lds[q * kWideThreads + tid];
                else xq = make_float4(xr[q][0], xr[q][1], xr[q][2], xr[q][3]);
                if constexpr (RAGGED) {                        // a straddling quad: its foreign columns are zero
                    if (dup[q] > 0) av[r][q].x = 0.f;
                    if (dup[q] > 1) av[r][q].y = 0.f;
                    if (dup[q] > 2) av[r][q].z = 0.f;
                }
                float p = fmaf(av[r][q].x, xq.x, s);
                p = fmaf(av[r][q].y, xq.y, p);
                p = fmaf(av[r][q].z, xq.z, p);
                p = fmaf(av[r][q].w, xq.w, p);
                s = dup[q] < 4 ? p : s;
            }
            s = group_sum<kWave>(s);
            if (lane == 0) sums[buf][r][wave] = s;
        }
        __syncthreads();           // two buffers: the next group's sums are written to the other one
        float coef[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < kWideWaves; ++w) s += sums[buf][r][w];
            coef[r] = live[r] ? loss_derivative(yl[r], s, loss) : 0.f;
        }
        // the group's rows are added to one another first: a shorter chain of additions per column
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if constexpr (R == 1) {
                acc[q][0] = fmaf(coef[0], av[0][q].x, acc[q][0]);
                acc[q][1] = fmaf(coef[0], av[0][q].y, acc[q][1]);
                acc[q][2] = fmaf(coef[0], av[0][q].z, acc[q][2]);
                acc[q][3] = fmaf(coef[0], av[0][q].w, acc[q][3]);
            } else {
                float g[4] = {coef[0] * av[0][q].x, coef[0] * av[0][q].y, coef[0] * av[0][q].z, coef[0] * av[0][q].w};
#pragma unroll
                for (int r = 1; r < R; ++r) {
                    g[0] = fmaf(coef[r], av[r][q].x, g[0]);
                    g[1] = fmaf(coef[r], av[r][q].y, g[1]);
                    g[2] = fmaf(coef[r], av[r][q].z, g[2]);
                    g[3] = fmaf(coef[r], av[r][q].w, g[3]);
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[q][t] += g[t];
            }
        }
        const bool end_of_chunk = l + R >= l1 || (kChunks > 1 && l + R == (chunk + 1) * rows_per_chunk);
        if (kFold && (++unfolded == kFoldGroups || end_of_chunk)) {
            unfolded = 0;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                float4 f = folded[q * kWideThreads + tid];
                f.x += acc[q][0];
                f.y += acc[q][1];
                f.z += acc[q][2];
                f.w += acc[q][3];
                folded[q * kWideThreads + tid] = f;
                const float back[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[q][t] = end_of_chunk ? back[t] : 0.f;
            }
        }
        if (end_of_chunk) {
            float *out = part + (worker * chunks + chunk) * d;
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (t >= dup[q]) out[at[q] + t] = acc[q][t];
                    acc[q][t] = 0.f;
                }
            ++chunk;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) av[r][q] = next[r][q];
            yl[r] = y_next[r];
            live[r] = live_next[r];
        }
    }
}

// Rows of a worker are cut so that all workers together have about one workgroup per compute unit, at least four
// rows each (a chunk's partial sums cost as much traffic as one of its rows, written and read again).  Never more
// chunks per worker than the partial sums have room for (max_chunks).
DensePlan wide_plan(int32_t n, int64_t m, int chunks_per_wg) {
    int64_t target = 256 / n;
    if (target < 1) target = 1;
    target *= chunks_per_wg;
    if (target > max_chunks(n, m)) target = max_chunks(n, m);
    int64_t rows = (m + target - 1) / target;
    if (rows < 4) rows = 4;
    return {rows, (m + rows - 1) / rows};
}

// ------------------------------------------------------------------ dense, any d: two passes
__global__ __launch_bounds__(kThreads) void logreg_dense_residual_kernel(const float *__restrict__ A,
                                                                         const float *__restrict__ y,
                                                                         const float *__restrict__ x,
                                                                         float *__restrict__ r, int64_t rows,
                                                                         int64_t d, int loss, int64_t m,
                                                                         const int32_t *__restrict__ batch,
                                                                         int64_t m_full, int64_t x_stride) {
    const int lane = lane_id();
    const int64_t nwaves = (int64_t)gridDim.x * kWaves;
    for (int64_t l = (int64_t)blockIdx.x * kWaves + threadIdx.x / kWave; l < rows; l += nwaves) {
        int64_t src = l;                        // rows counts n * m entries; with a batch, m of m_full rows each
        if (batch) {
            const int64_t b = batch_row(batch, l, m_full);
            if (b < 0) {
                if (lane == 0) r[l] = 0.f;
                continue;
            }
            src = (l / m) * m_full + b;
        }
        const float *row = A + src * d;
        const float *xw = x + (l / m) * x_stride;
        float s = 0.f;
        for (int64_t c = lane; c < d; c += kWave) s = fmaf(row[c], xw[c], s);
        s = wave_sum(s);
        if (lane == 0) r[l] = loss_derivative(y[src], s, loss);
    }
}

__global__ __launch_bounds__(kThreads) void logreg_dense_atr_kernel(const float *__restrict__ A,
                                                                    const float *__restrict__ r,
                                                                    float *__restrict__ part, int64_t m, int64_t d,
                                                                    int64_t rows_per_wg,
                                                                    const int32_t *__restrict__ batch,
                                                                    int64_t m_full) {
    const int64_t worker = blockIdx.z, chunk = blockIdx.y, chunks = gridDim.y;
    const int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (c >= d) return;
    const int64_t l0 = chunk * rows_per_wg;
    const int64_t l1 = l0 + rows_per_wg < m ? l0 + rows_per_wg : m;
    float acc = 0.f;
    for (int64_t l = l0; l < l1; ++l) {
        int64_t src = l;
        if (batch) {
            src = batch_row(batch, worker * m + l, m_full);
            if (src < 0) continue;              // its residual is zero as well
        }
        acc = fmaf(r[worker * m + l], A[(worker * m_full + src) * d + c], acc);
    }
    part[(worker * chunks + chunk) * d + c] = acc;
}

// grad[i][j] from the partial sums: one thread per (worker, column).
__global__ __launch_bounds__(kThreads) void logreg_dense_finish_kernel(const float *__restrict__ part,
                                                                       const float *__restrict__ x,
                                                                       float *__restrict__ grad, int64_t chunks,
                                                                       int64_t m, int64_t d, float lambda,
                                                                       int64_t x_stride) {
    const int64_t worker = blockIdx.y;
    const int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (c < d)
        grad[worker * d + c] =
            dense_grad_entry(part + worker * chunks * d, chunks, d, c, x[worker * x_stride + c], m, lambda);
}

// The same where a column has many sums: eight threads per column, a chain of dense_grad_entry's each, and all of a chain's
// entries in flight up to AHEAD of them (in memory order a thread alone waits for every sixteen: 12.8 us of a gradient's 26 at n = 1,
// m = 200000, d = 80 with 512 blocks).
constexpr int kSharedCols = 64, kSharedThreads = 8 * kSharedCols;
template <int AHEAD>
__global__ __launch_bounds__(kSharedThreads) void logreg_dense_finish_shared_kernel(const float *__restrict__ part,
                                                                                   const float *__restrict__ x,
                                                                                   float *__restrict__ grad,
                                                                                   int64_t chunks, int64_t m, int64_t d,
                                                                                   float lambda, int64_t x_stride) {
    __shared__ double lds[8 * kSharedCols];
    const int64_t worker = blockIdx.y;
    dense_grad_shared<kSharedThreads, kSharedCols, AHEAD>(part + worker * chunks * d, chunks, d,
                                                          (int64_t)blockIdx.x * kSharedCols, x + worker * x_stride, m, lambda,
                                                          lds, [&](int c, float g) { grad[worker * d + c] = g; });
}

struct DenseArgs {
    const float *A, *y, *x;
    float *part;
    int32_t n;
    int64_t m, d;          // m: rows summed per worker (the batch size under a batch)
    DensePlan pl;
    int loss;
    const int32_t *batch;
    int64_t m_full, x_stride;
    bool deep;
};

template <int LANES, int NQ, bool DEEP, int SHAPE>
void launch_fused_rows(const DenseArgs &a, hipStream_t stream) {
    const dim3 grid((unsigned)a.pl.chunks, (unsigned)a.n);
    if (a.batch)
        hipLaunchKernelGGL((logreg_dense_fused_kernel<LANES, NQ, DEEP, SHAPE, true>), grid, dim3(kThreads), 0, stream, a.A,
                           a.y, a.x, a.part, a.m, a.d, a.pl.rows_per_wg, a.loss, a.batch, a.m_full, a.x_stride);
    else
        hipLaunchKernelGGL((logreg_dense_fused_kernel<LANES, NQ, DEEP, SHAPE, false>), grid, dim3(kThreads), 0, stream, a.A,
                           a.y, a.x, a.part, a.m, a.d, a.pl.rows_per_wg, a.loss, a.batch, a.m_full, a.x_stride);
}

template <int LANES, int NQ>
void launch_fused(const DenseArgs &a, hipStream_t stream) {
    const bool quads = a.d % 4 == 0;
    if constexpr (NQ < 8) {
        if (a.deep) {
            if (quads) launch_fused_rows<LANES, NQ, true, kQuadRows>(a, stream);
            else launch_fused_rows<LANES, NQ, true, kRaggedRows>(a, stream);
            return;
        }
    }
    if (quads) launch_fused_rows<LANES, NQ, false, kQuadRows>(a, stream);
    else launch_fused_rows<LANES, NQ, false, kRaggedRows>(a, stream);
}

template <int NQ, bool RAGGED>
void launch_wide_tile(const DenseArgs &a, hipStream_t stream) {
    constexpr int64_t kChunks = wide_chunks<NQ>();
    const dim3 grid((unsigned)((a.pl.chunks + kChunks - 1) / kChunks), (unsigned)a.n);
    if (a.batch)
        hipLaunchKernelGGL((logreg_dense_wide_kernel<NQ, RAGGED, true>), grid, dim3(kWideThreads), 0, stream, a.A, a.y,
                           a.x, a.part, a.m, a.d, a.pl.rows_per_wg, a.pl.chunks, a.loss, a.batch, a.m_full, a.x_stride);
    else
        hipLaunchKernelGGL((logreg_dense_wide_kernel<NQ, RAGGED, false>), grid, dim3(kWideThreads), 0, stream, a.A, a.y,
                           a.x, a.part, a.m, a.d, a.pl.rows_per_wg, a.pl.chunks, a.loss, a.batch, a.m_full, a.x_stride);
}

template <int NQ>
void launch_wide(const DenseArgs &a, hipStream_t stream) {
    if (a.d % 4 == 0) launch_wide_tile<NQ, false>(a, stream);
    else launch_wide_tile<NQ, true>(a, stream);
}

}  // namespace

size_t logreg_dense_scratch_bytes(int32_t n, int64_t m, int64_t d) {
    return sizeof(float) * ((size_t)n * max_chunks(n, m) * d + (size_t)n * m);   // partial sums + residuals
}

hipError_t launch_logreg_grad_dense(const float *A, const float *y, const float *x, float *grad, int32_t n,
                                    int64_t m_full, int64_t d, float lambda, void *scratch, hipStream_t stream,
                                    const Marker &mk, GradParts *defer, int loss, RowBatch rb, int64_t x_stride,
                                    int64_t few_cols) {
    if (defer) *defer = GradParts();
    const int32_t *batch = rb.tau > 0 ? rb.rows : nullptr;
    const int64_t m = batch ? rb.tau : m_full;         // rows summed per worker (tau <= m_full, checked by the caller)
    if (solo_applies(n, m, m_full, d)) {
        const hipError_t st = launch_solo_grad(A, y, x, grad, n, m_full, d, lambda, loss, rb, x_stride, stream);
        mk(K_GRAD_MAIN);
        return st;
    }
    const DenseVariant dv = dense_variant(d);
    const bool deep = dense_deep(n, m_full, d) && d >= 4;
    const bool wide = dv.lanes == 0 && d <= kWideMax && d >= 4;
    const DensePlan pl = wide ? wide_plan(n, m, d > 4 * 4 * kWideThreads ? wide_chunks<5>() : wide_chunks<4>())
                              : dense_plan(n, m, d, deep);
    float *part = (float *)scratch;
    float *resid = part + (size_t)n * max_chunks(n, m_full) * d;
    const DenseArgs a{A, y, x, part, n, m, d, pl, loss, batch, m_full, x_stride, deep};
    const bool fused = dv.lanes != 0 || wide;
    switch (dv.lanes * 100 + dv.nq) {
        case 1601:
            if (d < 4) launch_fused_rows<16, 1, false, kTinyRows>(a, stream);
            else launch_fused<16, 1>(a, stream);
            break;
        case 3201: launch_fused<32, 1>(a, stream); break;
        case 6401: launch_fused<64, 1>(a, stream); break;
        case 6402: launch_fused<64, 2>(a, stream); break;
        case 6404: launch_fused<64, 4>(a, stream); break;
        case 6408: launch_fused<64, 8>(a, stream); break;
        case 6416: launch_fused_rows<64, 16, false, kQuadRows>(a, stream); break;
        default: break;
    }
    if (wide) {
        switch ((d + 4 * kWideThreads - 1) / (4 * kWideThreads)) {
            case 1: launch_wide<1>(a, stream); break;
            case 2: launch_wide<2>(a, stream); break;
            case 3: launch_wide<3>(a, stream); break;
            case 4: launch_wide<4>(a, stream); break;
            case 5: launch_wide<5>(a, stream); break;
            case 6: launch_wide<6>(a, stream); break;
            default: launch_wide<7>(a, stream); break;
        }
    }
    if (!fused) {
        const int64_t rows = (int64_t)n * m;
        int64_t blocks = (rows + kWaves - 1) / kWaves;
        if (blocks > 16384) blocks = 16384;
        hipLaunchKernelGGL(logreg_dense_residual_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, stream, A, y, x,
                           resid, rows, d, loss, m, batch, m_full, x_stride);
        hipLaunchKernelGGL(logreg_dense_atr_kernel,
                           dim3((unsigned)((d + kThreads - 1) / kThreads), (unsigned)pl.chunks, (unsigned)n),
                           dim3(kThreads), 0, stream, A, resid, part, m, d, pl.rows_per_wg, batch, m_full);
    }
    mk(K_GRAD_MAIN);
    hipError_t st = hipGetLastError();
    if (st != hipSuccess) return st;
    // The consumer finishes the sums itself (dense_grad_entry) where that is less work for its one workgroup per row than
    // another kernel of 3 to 5 us: on short rows (kRowPartsCols, kRowPartsFew) with few sums per column, or with more of them 1 us per 40 KB of
    // sums and per 1000 columns (the regulariser's divisions); many sums per column
    // go better by the threads of the kernel that shares them out.  step, us, with the sums left and finished: n = 2, m = 40000,
    // d = 250 (256 blocks) 31.3 and 27.2; n = 2, m = 50000, d = 300 (256) 34.6 and 31.5; n = 1, m = 200000, d = 80 (512) 26.8 and
    // 25.5.
    constexpr int64_t kColumnWork = 25, kFewBlocks = 32, kPartsWork = 60000, kPartsBlocks = 256;
    const bool little = pl.chunks <= kFewBlocks || (pl.chunks <= kPartsBlocks && (pl.chunks + kColumnWork) * d <= kPartsWork);
    const bool left = d <= kRowPartsCols ? little : pl.chunks <= kRowPartsFew && d <= few_cols && d <= kRowPartsMax;
    if (defer && fused && x_stride == 0 && left) {
        *defer = GradParts{part, pl.chunks, m, x, lambda};
        return hipSuccess;
    }
    const dim3 shared_grid((unsigned)((d + kSharedCols - 1) / kSharedCols), (unsigned)n);
    // Up to sixteen sums are one round trip of a thread alone, a chain of up to eight is one of a shared column's.  Enough columns
    // fill the chip by themselves (n = 8, m = 2000, d = 12000, 32 sums: 124.0 us the gradient by a thread per column, 125.0 shared;
    // n = 10, m = 5000, d = 1000, 51 sums: 35.3 and 34.3).
    constexpr int64_t kAloneMost = 16, kFewMost = 64, kFewColumns = 32768;
    const bool alone = pl.chunks <= kAloneMost || (pl.chunks <= kFewMost && (int64_t)n * d > kFewColumns);
    if (!alone && pl.chunks <= kFewMost)
        hipLaunchKernelGGL(logreg_dense_finish_shared_kernel<8>, shared_grid, dim3(kSharedThreads), 0, stream, part, x, grad,
                           pl.chunks, m, d, lambda, x_stride);
    else if (!alone)
        hipLaunchKernelGGL(logreg_dense_finish_shared_kernel<16>, shared_grid, dim3(kSharedThreads), 0, stream, part, x, grad,
                           pl.chunks, m, d, lambda, x_stride);
    else
        hipLaunchKernelGGL(logreg_dense_finish_kernel, dim3((unsigned)((d + kThreads - 1) / kThreads), (unsigned)n),
                           dim3(kThreads), 0, stream, part, x, grad, pl.chunks, m, d, lambda, x_stride);
    mk(K_GRAD_AUX);
    return hipGetLastError();
}

}  // namespace ef21
