// Vector kernels of Algorithm 2: the model step (line 3), the master's aggregation of the messages
// (line 8), and the mean of the workers' estimators (input line, g^0 = (1/n) sum_i g_i^0).
#include <algorithm>
#include <type_traits>

#include "device_utils.h"
#include "kernels.h"

namespace ef21 {
namespace {

constexpr int kThreads = 256;
// Past the caches a block copies 2048 entries, through them a block per compute unit its share (copy_way.h says which).
constexpr int kCopyThreads = 512, kCopyBlocks = 256;

// x_j <- x_j - gamma g_j as one fused multiply-add per coordinate (a single rounding).
__global__ __launch_bounds__(kThreads) void model_step_kernel(float *__restrict__ x, const float *__restrict__ g,
                                                              int64_t d, float neg_gamma) {
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    for (int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x; j < d; j += stride)
        x[j] = fmaf(neg_gamma, g[j], x[j]);
}

// Same, four coordinates per lane; needs d % 4 == 0 and 16-byte aligned pointers.
__global__ __launch_bounds__(kThreads) void model_step_vec4_kernel(float4 *__restrict__ x,
                                                                   const float4 *__restrict__ g, int64_t d4,
                                                                   float neg_gamma) {
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    for (int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x; j < d4; j += stride) {
        float4 xv = x[j];
        const float4 gv = g[j];
        xv.x = fmaf(neg_gamma, gv.x, xv.x);
        xv.y = fmaf(neg_gamma, gv.y, xv.y);
        xv.z = fmaf(neg_gamma, gv.z, xv.z);
        xv.w = fmaf(neg_gamma, gv.w, xv.w);
        x[j] = xv;
    }
}

// The rows' mean, and on the way a copy of the rows (rows_out) and of one more vector (x_out <- x) for ef21_set_state, which
// took a launch each and read the rows twice.  Per coordinate the workers in order, in fp64, rounded once.  FLIGHT workers' loads
// in flight: up to eight where a thread has four columns, up to 32 where it has one: short rows have few threads, and there the waits for memory
// are all there is (20 x 123, the three things in 4 launches 9.4 us, in this one 3.0; with 32 for any number of workers, the last one's read again,
// 2 x 2000 took 2.9 against 2.0 and the mean alone 0.9 more than the kernel before).  Rows may start at any 4-byte address.
struct RowsOut {
    float *rows;                 // nullptr: the mean alone
    const float *x;              // with x_out, or nullptr
    float *x_out;
};
enum RowsCopy { kNoCopy = 0, kCopy = 1, kCopyStreamed = 2, kNoCopyStreamed = 3 };      // streamed: past the caches, see mean_way
template <int VEC, int COPY, int FLIGHT>
__global__ __launch_bounds__(kThreads) void mean_rows_kernel(const float *__restrict__ g_i, float *__restrict__ g,
                                                             int32_t n, int64_t d, RowsOut out) {
    const int64_t stride = (int64_t)gridDim.x * kThreads * VEC;
    auto columns = [&](auto width, int64_t j) {
        constexpr int W = decltype(width)::value;
        double s[W] = {};
        for (int32_t i0 = 0; i0 < n; i0 += FLIGHT) {
            float v[FLIGHT][W];
#pragma unroll
            for (int u = 0; u < FLIGHT; ++u) {      // a worker past the end re-reads the last one, unused
                const float *at = g_i + (int64_t)(i0 + u < n ? i0 + u : n - 1) * d + j;
                if constexpr (W == 4) {
                    const float4 t = COPY != kNoCopy ? stream_load4_any(at) : load4_any(at);
                    v[u][0] = t.x, v[u][1] = t.y, v[u][2] = t.z, v[u][3] = t.w;
                } else {
                    v[u][0] = *at;
                }
            }
#pragma unroll
            for (int u = 0; u < FLIGHT; ++u) {
                if (i0 + u < n) {
#pragma unroll
                    for (int t = 0; t < W; ++t) s[t] += (double)v[u][t];
                    if constexpr (COPY == kCopy || COPY == kCopyStreamed) {
                        float *to = out.rows + (int64_t)(i0 + u) * d + j;
                        if constexpr (W != 4) *to = v[u][0];
                        else if constexpr (COPY == kCopyStreamed) stream_store4_any(to, make_float4(v[u][0], v[u][1], v[u][2], v[u][3]));
                        else store4_any(to, make_float4(v[u][0], v[u][1], v[u][2], v[u][3]));
                    }
                }
            }
        }
#pragma unroll
        for (int t = 0; t < W; ++t) {
            g[j + t] = (float)(s[t] / (double)n);
            if ((COPY == kCopy || COPY == kCopyStreamed) && out.x_out) out.x_out[j + t] = out.x[j + t];
        }
    };
    for (int64_t j = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * VEC; j < d; j += stride) {
        if (j + VEC <= d) columns(std::integral_constant<int, VEC>(), j);
        else
            for (int64_t c = j; c < d; ++c) columns(std::integral_constant<int, 1>(), c);
    }
}

// Up to three arrays copied by one launch, 16 bytes a thread and access, at any 4-byte address.  STREAM: past the caches.
template <bool STREAM>
__global__ __launch_bounds__(kCopyThreads) void copy_arrays_kernel(CopyList c) {
    constexpr int kInFlight = 4;
    const int64_t stride = (int64_t)gridDim.x * kCopyThreads * 4;
    auto load = [](const float *p) { return STREAM ? stream_load4_any(p) : load4_any(p); };
    auto store = [](float *p, const float4 &v) {
        if constexpr (STREAM) stream_store4_any(p, v);
        else store4_any(p, v);
    };
    for (int a = 0; a < 3; ++a) {
        const float *src = c.src[a];
        float *dst = c.dst[a];
        const int64_t count = c.count[a];
        int64_t e = ((int64_t)blockIdx.x * kCopyThreads + threadIdx.x) * 4;
        for (; e + (kInFlight - 1) * stride + 4 <= count; e += kInFlight * stride) {
            float4 v[kInFlight];
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) v[u] = load(src + e + u * stride);
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) store(dst + e + u * stride, v[u]);
        }
        for (; e < count; e += stride) {
            if (e + 4 <= count) store(dst + e, load(src + e));
            else
                for (int64_t t = e; t < count; ++t) dst[t] = src[t];
        }
    }
}

// ---- Algorithm 2, line 8 (and line 3) without atomics ------------------------------------------
// The coordinates are cut into sub-blocks of kAggSub.  A worker's message is sorted by position, so
// its entries inside a sub-block are one contiguous run [start[w][b], start[w][b+1]); the runs are
// recorded by message_index_kernel.  aggregate_kernel gives each sub-block to ONE wavefront, which
// adds the workers' runs one after the other into its LDS accumulator (positions inside a message are
// distinct, so a plain read-add-write is enough, and a single wavefront needs no barrier between
// workers): the sum runs in worker order, g is bitwise reproducible, and no global atomic is issued.
constexpr int kAggSub = 512, kAggLong = 2048;      // columns of a sub-block; see aggregate_kernel
constexpr int kAggWaves = kThreads / kWave;

// A thread per entry of the message.
__global__ __launch_bounds__(kThreads) void message_index_kernel(const int32_t *__restrict__ idx, int64_t k,
                                                                 int64_t nblk, int32_t sub,
                                                                 int32_t *__restrict__ start) {
    const int64_t w = blockIdx.y;
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p >= k) return;
    const int32_t *row = idx + w * k;
    int32_t *out = start + w * (nblk + 1);
    const int64_t b_cur = row[p] / sub;
    const int64_t b_prev = p > 0 ? row[p - 1] / sub : -1;
    for (int64_t b = b_prev + 1; b <= b_cur; ++b) out[b] = (int32_t)p;     // first entry of sub-block b
    if (p == k - 1)
        for (int64_t b = b_cur + 1; b <= nblk; ++b) out[b] = (int32_t)k;
}

// A thread per sub-block: the first entry at or beyond its first coordinate.
__global__ __launch_bounds__(kThreads) void message_index_search_kernel(const int32_t *__restrict__ idx, int64_t k,
                                                                        int64_t nblk, int32_t sub,
                                                                        int32_t *__restrict__ start) {
    const int64_t w = blockIdx.y;
    const int64_t b = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (b > nblk) return;
    const int32_t *row = idx + w * k;
    int64_t lo = 0, hi = b < nblk ? k : 0;                                 // start[nblk] = k
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if ((int64_t)row[mid] < b * sub) lo = mid + 1;
        else hi = mid;
    }
    start[w * (nblk + 1) + b] = (int32_t)(b < nblk ? lo : k);
}

// A thread per entry writes the starts of all sub-blocks since the entry before it: as many as there are, where a long
// row's message is one or a few entries (step of 2 rows of 10 million, k = 1: 612 us, 197 with blocks of 2048; 62 with a
// search per sub-block; 20 rows of a million 162 and 42).
void launch_message_index(const int32_t *idx, int32_t n, int64_t k, int64_t nblk, int32_t sub, int32_t *start,
                          hipStream_t stream) {
    const bool search = nblk > 4 * k;
    const dim3 grid((unsigned)(((search ? nblk + 1 : k) + kThreads - 1) / kThreads), (unsigned)n), block(kThreads);
    if (search) hipLaunchKernelGGL(message_index_search_kernel, grid, block, 0, stream, idx, k, nblk, sub, start);
    else hipLaunchKernelGGL(message_index_kernel, grid, block, 0, stream, idx, k, nblk, sub, start);
}

// The runs of workers [w_lo, w_hi) inside sub-block b (columns from c0) added to `acc`, worker after worker, by
// the calling wavefront.
__device__ __forceinline__ void add_runs(const int32_t *__restrict__ idx, const float *__restrict__ val,
                                         const int32_t *__restrict__ start, int64_t nblk, int64_t b, int64_t k,
                                         int32_t w_lo, int32_t w_hi, float *acc, int64_t c0, int lane) {
    constexpr int kInFlight = 8;                     // workers whose runs are loaded together
    for (int32_t w0 = w_lo; w0 < w_hi; w0 += kWave) {
        const int32_t w = w0 + lane;
        const int32_t s0 = w < w_hi ? start[(int64_t)w * (nblk + 1) + b] : 0;
        const int32_t s1 = w < w_hi ? start[(int64_t)w * (nblk + 1) + b + 1] : 0;
        const int32_t tile = w_hi - w0 < kWave ? w_hi - w0 : kWave;
        for (int32_t t0 = 0; t0 < tile; t0 += kInFlight) {
            int32_t e[kInFlight], len[kInFlight];
            int64_t base[kInFlight];
            float v[kInFlight];
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                const int src = t0 + u < tile ? t0 + u : 0;
                const int32_t lo = __shfl(s0, src, kWave), hi = __shfl(s1, src, kWave);
                len[u] = t0 + u < tile ? hi - lo : 0;
                base[u] = (int64_t)(w0 + src) * k + lo;
                const int64_t at = lane < len[u] ? base[u] + lane : 0;     // unconditional loads, no branch
                e[u] = idx[at];
                v[u] = val[at];
                if (lane >= len[u]) e[u] = -1;
            }
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {     // worker order
                if (e[u] >= 0) acc[e[u] - c0] += v[u];
                for (int32_t j = lane + kWave; j < len[u]; j += kWave) acc[idx[base[u] + j] - c0] += val[base[u] + j];
            }
        }
    }
}

// What bounds it: the bytes of g and x, provided the wavefront waits for memory once and not once per 256 columns, so
// g and x are fetched whole into registers before the runs are added, by enough wavefronts: blocks of 512 columns fill
// the chip from 10^5 columns on, and a worker's run fits the 64 lanes up to a tenth of the entries kept.  (Blocks of 2048
// without the prefetch: 18.4 us against 8.5 at d = 1000003, n = 5, k = 50000; 45.9 against 45.4 at d = 11.2 million, where
// the 180 MB of g and x at the rate of a plain copy take 39; blocks of 2048 with it: 50.)
// Where blocks of 2048 fill the chip as well and a run is a handful of entries, the longer blocks are the better ones: a
// quarter as many run bounds to read here and to write in the emission.  step, us, with 512 and 2048 columns: n = 15, d = 5
// million, k = 50000 178 and 174; n = 9, d = 4 million, k = 40000 101 and 97.5; n = 12, d = 6 million, k = 6000 138.5 and
// 134; n = 9, d = 8 million, k = 80000 181 and 175; but n = 15, d = 2 million, k = 20000 81 and 83.4; n = 15, d = 4.2 million,
// k = 210000 214 and 222; n = 8, d = 11.2 million, k = 112000 248 and 251 (with the copy of x that follows); n = 2, d = 40
// million, k = 400000 330 and 338.
// vec: g and x 16-byte aligned (a block starts at a multiple of 512 columns whatever d is); the last, partial block
// and unaligned vectors go column by column.
template <bool STEP, int SUB>
__global__ __launch_bounds__(kThreads) void aggregate_kernel(const int32_t *__restrict__ idx,
                                                             const float *__restrict__ val,
                                                             const int32_t *__restrict__ start, int32_t n, int64_t k,
                                                             int64_t d, int64_t nblk, float *__restrict__ g,
                                                             float *__restrict__ x, float inv_n, float neg_gamma,
                                                             bool vec, bool from_zero) {
    constexpr int kPer = SUB / (4 * kWave);
    constexpr bool kAhead = SUB == kAggSub;
    __shared__ __attribute__((aligned(16))) float lds[kAggWaves][SUB];
    const int wave = threadIdx.x / kWave, lane = lane_id();
    const int64_t b = (int64_t)blockIdx.x * kAggWaves + wave;
    if (b >= nblk) return;
    float *acc = lds[wave];
    const int64_t c0 = b * SUB;
    const int64_t c1 = c0 + SUB < d ? c0 + SUB : d;
    const bool whole = vec && c0 + SUB <= d;
    float4 g4[kAhead ? kPer : 1], x4[kAhead ? kPer : 1];
    auto fetch = [&](int q, float4 &gq, float4 &xq) {
        gq = make_float4(0.f, 0.f, 0.f, 0.f);
        if (!from_zero) gq = *reinterpret_cast<const float4 *>(g + c0 + 4 * (q * kWave + lane));
        if (STEP) xq = *reinterpret_cast<const float4 *>(x + c0 + 4 * (q * kWave + lane));
    };
    if constexpr (kAhead) {
        if (whole) {
#pragma unroll
            for (int q = 0; q < kPer; ++q) fetch(q, g4[q], x4[q]);
        }
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) *reinterpret_cast<float4 *>(acc + 4 * (q * kWave + lane)) = make_float4(0.f, 0.f, 0.f, 0.f);
    add_runs(idx, val, start, nblk, b, k, 0, n, acc, c0, lane);
    if (whole) {
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            float4 &gq = g4[kAhead ? q : 0], &xq = x4[kAhead ? q : 0];
            if constexpr (!kAhead) fetch(q, gq, xq);
            const float4 a4 = *reinterpret_cast<const float4 *>(acc + 4 * (q * kWave + lane));
            gq.x = fmaf(a4.x, inv_n, gq.x);
            gq.y = fmaf(a4.y, inv_n, gq.y);
            gq.z = fmaf(a4.z, inv_n, gq.z);
            gq.w = fmaf(a4.w, inv_n, gq.w);
            *reinterpret_cast<float4 *>(g + c0 + 4 * (q * kWave + lane)) = gq;
            if (STEP) {
                xq.x = fmaf(neg_gamma, gq.x, xq.x);
                xq.y = fmaf(neg_gamma, gq.y, xq.y);
                xq.z = fmaf(neg_gamma, gq.z, xq.z);
                xq.w = fmaf(neg_gamma, gq.w, xq.w);
                *reinterpret_cast<float4 *>(x + c0 + 4 * (q * kWave + lane)) = xq;
            }
        }
    } else {
        for (int64_t j = c0 + lane; j < c1; j += kWave) {
            const float gj = fmaf(acc[j - c0], inv_n, from_zero ? 0.f : g[j]);
            g[j] = gj;
            if (STEP) x[j] = fmaf(neg_gamma, gj, x[j]);
        }
    }
}

// Many workers (n >= kManyWorkers): the chain of n dependent additions per sub-block is what takes the time, so
// a workgroup of four wavefronts shares ONE sub-block of kManySub columns: wavefront j adds the j-th quarter of
// the workers (in worker order) into its own accumulator, and the four are then added in order,
// ((a0 + a1) + a2) + a3: a fixed association, so g stays bitwise reproducible.
constexpr int kManyWorkers = 16, kManySub = 256;
static_assert(kManySub == kThreads, "one column per thread in the last step");

template <bool STEP>
__global__ __launch_bounds__(kThreads) void aggregate_many_kernel(const int32_t *__restrict__ idx,
                                                                  const float *__restrict__ val,
                                                                  const int32_t *__restrict__ start, int32_t n,
                                                                  int64_t k, int64_t d, int64_t nblk,
                                                                  float *__restrict__ g, float *__restrict__ x,
                                                                  float inv_n, float neg_gamma, bool from_zero) {
    __shared__ float lds[kAggWaves][kManySub];
    const int wave = threadIdx.x / kWave, lane = lane_id();
    const int64_t b = blockIdx.x, c0 = b * kManySub;
    const int64_t j = c0 + threadIdx.x;
    const float gj = !from_zero && j < d ? g[j] : 0.f;       // fetched while the runs are added
    const float xj = STEP && j < d ? x[j] : 0.f;
    float *acc = lds[wave];
    for (int t = lane; t < kManySub; t += kWave) acc[t] = 0.f;
    const int32_t quarter = (n + kAggWaves - 1) / kAggWaves;
    const int32_t w_lo = wave * quarter < n ? wave * quarter : n;
    const int32_t w_hi = w_lo + quarter < n ? w_lo + quarter : n;
    add_runs(idx, val, start, nblk, b, k, w_lo, w_hi, acc, c0, lane);
    __syncthreads();
    if (j < d) {
        const float a = ((lds[0][threadIdx.x] + lds[1][threadIdx.x]) + lds[2][threadIdx.x]) + lds[3][threadIdx.x];
        const float gn = fmaf(a, inv_n, gj);
        g[j] = gn;
        if (STEP) x[j] = fmaf(neg_gamma, gn, xj);
    }
}

// Small problems (aggregate_is_small): one workgroup, one launch.  All threads stage the
// messages in LDS; then ONE wavefront adds them to the LDS accumulator worker by worker, 64 entries of a
// worker per step (positions inside a message are distinct, and a wavefront's LDS accesses execute in
// program order, so no barrier is needed between workers) while the other wavefronts fetch g and x.
// Room for what the rule admits, in two sizes: up to two pairs a thread and 12 288 columns, or up to eight pairs and 3072 columns.
// With eight and 16 384 for all calls a step of 4 x 1000, k = 100 took 8.6 us, of 1 x 622, k = 622 8.5 and of 64 x 70, k = 20 14.5: 8.1,
// 8.0 and 12.3 so.
constexpr int kSmallThreads = 1024;
constexpr int kFewPer = 2, kFewCols = 12288, kManyPer = 8, kManyCols = 3072;
constexpr int kSmallSteps = 512;     // at most this many sequential steps of the adding wavefront
constexpr int kScanEntries = 128;    // messages in all that every coordinate can look through (n = 20, k = 4: 4.8 -> 2.8 us)
constexpr int kSmallFetch = 4;       // coordinates per thread fetched ahead (d <= 4096)
// Steps whose pairs are in registers.  step with supplied gradients, us, one step ahead and eight: 20 x 1000, k = 100 13.1 and 12.2;
// 64 x 300, k = 30 14.8 and 13.7; 200 x 200, k = 10 32.6 and 27.3.
constexpr int kSmallAhead = 8;
// Pairs of a worker up to which an LDS atomic is the quicker addition.  The same, us, read-add-write and atomic: 500 x 256, k = 4
// 70.5 and 59.3; 64 x 300, k = 30 14.5 and 13.7; 8 x 1000, k = 64 8.1 and 8.4; 20 x 1000, k = 100 12.2 and 12.7.
constexpr int kSmallLanes = 32;

template <bool STEP, int PER, int COLS>
__global__ __launch_bounds__(kSmallThreads) void aggregate_small_kernel(const int32_t *__restrict__ idx,
                                                                        const float *__restrict__ val, int32_t n,
                                                                        int64_t k, int64_t d, float *__restrict__ g,
                                                                        float *__restrict__ x, float inv_n,
                                                                        float neg_gamma, bool from_zero) {
    __shared__ float acc[COLS];
    __shared__ __attribute__((aligned(16))) int32_t m_idx[PER * kSmallThreads];
    __shared__ __attribute__((aligned(16))) float m_val[PER * kSmallThreads];
    const int tid = threadIdx.x, lane = lane_id();
    const int64_t total = (int64_t)n * k;
    int32_t e[PER];
    float v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int64_t t = tid + (int64_t)u * kSmallThreads;
        const int64_t at = t < total ? t : 0;
        e[u] = idx[at];
        v[u] = val[at];
    }
    for (int64_t j = tid; j < d; j += kSmallThreads) acc[j] = 0.f;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int64_t t = tid + (int64_t)u * kSmallThreads;
        if (t < total) {
            m_idx[t] = e[u];
            m_val[t] = v[u];
        }
    }
    if (total <= kScanEntries && tid < 8) m_idx[total + tid] = -1;      // the scan below takes eight at a time
    __syncthreads();
    const bool ahead = d <= (int64_t)kSmallFetch * kSmallThreads;
    if (total <= kScanEntries && d <= kSmallThreads) {       // few messages: every coordinate looks through them all
        if (tid < d) {
            const float g0 = from_zero ? 0.f : g[tid], x0 = STEP ? x[tid] : 0.f;
            float a = 0.f;
            for (int t = 0; t < (int)total; t += 8) {        // eight at a time, in order: worker after worker
                const int4 i0 = *reinterpret_cast<const int4 *>(m_idx + t), i1 = *reinterpret_cast<const int4 *>(m_idx + t + 4);
                const float4 v0 = *reinterpret_cast<const float4 *>(m_val + t), v1 = *reinterpret_cast<const float4 *>(m_val + t + 4);
                a = i0.x == tid ? a + v0.x : a;
                a = i0.y == tid ? a + v0.y : a;
                a = i0.z == tid ? a + v0.z : a;
                a = i0.w == tid ? a + v0.w : a;
                a = i1.x == tid ? a + v1.x : a;
                a = i1.y == tid ? a + v1.y : a;
                a = i1.z == tid ? a + v1.z : a;
                a = i1.w == tid ? a + v1.w : a;
            }
            const float gn = fmaf(a, inv_n, g0);
            g[tid] = gn;
            if (STEP) x[tid] = fmaf(neg_gamma, gn, x0);
        }
        return;                                              // the whole workgroup
    }
    float gj[kSmallFetch], xj[kSmallFetch];
    if (tid < kWave) {
        // worker order; the pairs of eight steps (a worker's next 64 pairs each) are read before the first of them is added
        const int per = (int)((k + kWave - 1) / kWave), steps = n * per;
        int at = 0, i0 = 0;                         // of the next step: the worker's first pair, and how far into the message
        for (int s0 = 0; s0 < steps; s0 += kSmallAhead) {
            int32_t e8[kSmallAhead];
            float v8[kSmallAhead];
            bool in[kSmallAhead];
#pragma unroll
            for (int u = 0; u < kSmallAhead; ++u) {
                in[u] = s0 + u < steps && i0 + lane < k;
                const int from = in[u] ? at + i0 + lane : 0;
                e8[u] = m_idx[from];
                v8[u] = m_val[from];
                i0 += kWave;
                if (i0 >= k) {
                    i0 = 0;
                    at += (int)k;
                }
            }
#pragma unroll
            for (int u = 0; u < kSmallAhead; ++u) {
                if (in[u]) {
                    if (k <= kSmallLanes) lds_add(acc + e8[u], v8[u]);
                    else acc[e8[u]] += v8[u];
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
    if (ahead) {
#pragma unroll
        for (int u = 0; u < kSmallFetch; ++u) {
            const int64_t j = tid + (int64_t)u * kSmallThreads;
            gj[u] = !from_zero && j < d ? g[j] : 0.f;
            xj[u] = STEP && j < d ? x[j] : 0.f;
        }
    }
    __syncthreads();
    if (ahead) {
#pragma unroll
        for (int u = 0; u < kSmallFetch; ++u) {
            const int64_t j = tid + (int64_t)u * kSmallThreads;
            if (j < d) {
                const float gn = fmaf(acc[j], inv_n, gj[u]);
                g[j] = gn;
                if (STEP) x[j] = fmaf(neg_gamma, gn, xj[u]);
            }
        }
    } else {
        for (int64_t j = tid; j < d; j += kSmallThreads) {
            const float gn = fmaf(acc[j], inv_n, from_zero ? 0.f : g[j]);
            g[j] = gn;
            if (STEP) x[j] = fmaf(neg_gamma, gn, x[j]);
        }
    }
}

// ---- plain streaming kernels (measurement only): 2048 workgroups, each thread strides over the buffer
__global__ __launch_bounds__(kThreads) void hbm_read_kernel(const float *__restrict__ src, int64_t n16,
                                                            float *__restrict__ sink) {
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    float acc = 0.f;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n16; i += stride) {
        const float4 v = stream_load4(src + 4 * i);
        acc += (v.x + v.y) + (v.z + v.w);
    }
    acc = wave_sum(acc);
    if (acc == 1.2345e-31f) sink[0] = acc;       // keeps the loads alive; practically never stores
}

__global__ __launch_bounds__(kThreads) void hbm_copy_kernel(float4 *__restrict__ dst, const float4 *__restrict__ src,
                                                            int64_t n16) {
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

unsigned grid_for(int64_t items, int64_t cap) {
    int64_t blocks = (items + kThreads - 1) / kThreads;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return (unsigned)blocks;
}

}  // namespace

hipError_t launch_model_step(float *x, const float *g, int64_t d, float gamma, hipStream_t stream) {
    const bool vec = (d % 4 == 0) && (((uintptr_t)x | (uintptr_t)g) % 16 == 0);
    if (vec) {
        hipLaunchKernelGGL(model_step_vec4_kernel, dim3(grid_for(d / 4, 8192)), dim3(kThreads), 0, stream,
                           (float4 *)x, (const float4 *)g, d / 4, -gamma);
    } else {
        hipLaunchKernelGGL(model_step_kernel, dim3(grid_for(d, 8192)), dim3(kThreads), 0, stream, x, g, d,
                           -gamma);
    }
    return hipGetLastError();
}

size_t aggregate_index_bytes(int32_t n, int64_t d) {      // for the shorter of the two sub-block lengths
    return sizeof(int32_t) * (size_t)n * ((size_t)((d + kManySub - 1) / kManySub) + 1);
}

namespace {
// One workgroup adds one step (64 pairs of a worker) after the other, 0.12 us each, and walks all coordinates; the kernels with a
// wavefront or four per block of coordinates take a message index, which launch_topk_row_reg and launch_topk_split write with the
// message, and a kernel of its own (2.5 us) where neither selects, on short rows and where more than an eighth of a row is kept:
// there a block's runs are long, and their pairs are read in turn.  step with supplied gradients, us, small and not, workers x
// columns, k (steps + columns / 512).  With the index at hand: 5 x 10000, 30 (24) 10.4 and 10.4; 8 x 10000, 30 (27) 10.6 and 10.3;
// 10 x 5000, 130 (39) 12.4 and 11.6; 8 x 2000, 200 (35) 11.6 and 10.4.  Without: 8 x 300, 300 (40) 12.1 and 18.5; 12 x 500, 500 (96)
// 18.5 and 35.0; 4 x 1000, 1000 (65) 15.5 and 18.1; 2 x 1500, 1500 (50) 13.6 and 15.1; 15 x 1500, 195 (62) 16.2 and 14.7; 3 x 1500,
// 1500 (74) 17.1 and 16.8; 4 x 2468, 493 (36) 13.0 and 14.0; 6 x 2500, 325 (40) 14.5 and 13.6; 1 x 2500, 2500 (44) 13.4 and 14.6;
// 3 x 4000, 520 (34) 14.7 and 14.6; 1 x 8000, 2000 (47) 19.1 and 17.8; 16 workers and more: 16 x 300, 300 17.0 and 13.9; 32 x 500, 65
// 15.2 and 10.9.  Up to 1024 coordinates and 2048 pairs
// the sums are those of the iteration in one launch (small_step.hip) to the bit, in worker order, so they stay here.
constexpr int64_t kSmallStep1 = 1024, kReachIndexed = 24, kReachNot = 38, kReachNot1 = 44, kReachNot3 = 52, kSmallCols3 = 1536;
static_assert(kReachIndexed <= kReachNot, "with an index there is one more reason against the one workgroup");
bool aggregate_is_small(int32_t n, int64_t k, int64_t d, bool indexed) {
    const int64_t pairs = (int64_t)n * k, steps = (int64_t)n * ((k + kWave - 1) / kWave), reach = steps + d / 512;
    if (pairs > (int64_t)kManyPer * kSmallThreads || steps > kSmallSteps || d > kFewCols) return false;
    const bool few = pairs <= (int64_t)kFewPer * kSmallThreads;
    if (few && d <= kSmallStep1) return true;
    if (n >= kManyWorkers || !(few || d <= kManyCols)) return false;
    if (indexed) return reach <= kReachIndexed;
    return d <= kSmallStep1 || reach <= (d <= kSmallCols3 ? kReachNot3 : n == 1 ? kReachNot1 : kReachNot);
}
}  // namespace

int aggregate_index_shift(int32_t n, int64_t k, int64_t d) {
    static_assert(kManySub == 1 << 8 && kAggSub == 1 << 9 && kAggLong == 1 << 11, "block lengths as shifts");
    if (aggregate_is_small(n, k, d, true)) return -1;
    if (n >= kManyWorkers) return 8;
    return d >= 4000000 && d <= 8000000 && k * 100 <= d ? 11 : 9;
}

hipError_t launch_aggregate(const int32_t *idx, const float *val, int32_t n, int64_t k, int64_t d, float *g, float *x,
                            float gamma, void *index, hipStream_t stream, bool index_ready, bool from_zero) {
    const float inv_n = 1.0f / (float)n;
    if (!index_ready && aggregate_is_small(n, k, d, false)) {
#define EF21_SMALL(STEP, PER, COLS)                                                                                     \
    hipLaunchKernelGGL((aggregate_small_kernel<STEP, PER, COLS>), dim3(1), dim3(kSmallThreads), 0, stream, idx, val, n, k, \
                       d, g, x, inv_n, -gamma, from_zero)
        if ((int64_t)n * k <= (int64_t)kFewPer * kSmallThreads) {
            if (x) EF21_SMALL(true, kFewPer, kFewCols);
            else EF21_SMALL(false, kFewPer, kFewCols);
        } else {
            if (x) EF21_SMALL(true, kManyPer, kManyCols);
            else EF21_SMALL(false, kManyPer, kManyCols);
        }
#undef EF21_SMALL
        return hipGetLastError();
    }
    int32_t *start = (int32_t *)index;
    if (n >= kManyWorkers) {
        const int64_t nblk = (d + kManySub - 1) / kManySub;
        if (!index_ready) launch_message_index(idx, n, k, nblk, kManySub, start, stream);
        if (x)
            hipLaunchKernelGGL(aggregate_many_kernel<true>, dim3((unsigned)nblk), dim3(kThreads), 0, stream, idx, val,
                               start, n, k, d, nblk, g, x, inv_n, -gamma, from_zero);
        else
            hipLaunchKernelGGL(aggregate_many_kernel<false>, dim3((unsigned)nblk), dim3(kThreads), 0, stream, idx, val,
                               start, n, k, d, nblk, g, x, inv_n, -gamma, from_zero);
        return hipGetLastError();
    }
    const int shift = aggregate_index_shift(n, k, d);
    const int64_t nblk = ((d - 1) >> shift) + 1;
    if (!index_ready) launch_message_index(idx, n, k, nblk, 1 << shift, start, stream);
    const dim3 grid((unsigned)((nblk + kAggWaves - 1) / kAggWaves)), block(kThreads);
    const bool vec = ((uintptr_t)g | (uintptr_t)(x ? x : g)) % 16 == 0;
#define EF21_AGG(STEP, SUB)                                                                                              \
    hipLaunchKernelGGL((aggregate_kernel<STEP, SUB>), grid, block, 0, stream, idx, val, start, n, k, d, nblk, g, x, inv_n, \
                       -gamma, vec, from_zero)
    if (shift == 11 && x) EF21_AGG(true, kAggLong);
    else if (shift == 11) EF21_AGG(false, kAggLong);
    else if (x) EF21_AGG(true, kAggSub);
    else EF21_AGG(false, kAggSub);
#undef EF21_AGG
    return hipGetLastError();
}

hipError_t launch_hbm_read(const void *src, int64_t n16, float *sink, hipStream_t stream) {
    hipLaunchKernelGGL(hbm_read_kernel, dim3(grid_for(n16, 2048)), dim3(kThreads), 0, stream, (const float *)src, n16,
                       sink);
    return hipGetLastError();
}

hipError_t launch_hbm_copy(void *dst, const void *src, int64_t n16, hipStream_t stream) {
    hipLaunchKernelGGL(hbm_copy_kernel, dim3(grid_for(n16, 8192)), dim3(kThreads), 0, stream, (float4 *)dst,
                       (const float4 *)src, n16);
    return hipGetLastError();
}

hipError_t launch_mean_rows(const float *g_i, float *g, int32_t n, int64_t d, hipStream_t stream, float *rows_out,
                            const float *x, float *x_out) {
    const RowsOut out{rows_out, x, x_out};
    const MeanWay way = mean_way(n, d, rows_out != nullptr);
#define EF21_MEAN(VEC, COPY, FLIGHT)                                                                                    \
    hipLaunchKernelGGL((mean_rows_kernel<VEC, COPY, FLIGHT>), dim3(grid_for((d + VEC - 1) / VEC, 8192)), dim3(kThreads), 0, stream, \
                       g_i, g, n, d, out)
#define EF21_MEAN4(COPY) \
    do { \
        if (n <= 2) EF21_MEAN(4, COPY, 2); \
        else if (n <= 4) EF21_MEAN(4, COPY, 4); \
        else EF21_MEAN(4, COPY, 8); \
    } while (0)
#define EF21_MEAN1(COPY) \
    do { \
        if (n <= 2) EF21_MEAN(1, COPY, 2); \
        else if (n <= 4) EF21_MEAN(1, COPY, 4); \
        else if (n <= 8) EF21_MEAN(1, COPY, 8); \
        else if (n <= 16) EF21_MEAN(1, COPY, 16); \
        else EF21_MEAN(1, COPY, 32); \
    } while (0)
    if (way == MeanWay::kColumn && rows_out) EF21_MEAN1(kCopy);
    else if (way == MeanWay::kColumn) EF21_MEAN1(kNoCopy);
    else if (way == MeanWay::kQuadStreamed && rows_out) EF21_MEAN4(kCopyStreamed);
    else if (way == MeanWay::kQuadStreamed) EF21_MEAN4(kNoCopyStreamed);
    else if (rows_out) EF21_MEAN4(kCopy);
    else EF21_MEAN4(kNoCopy);
#undef EF21_MEAN1
#undef EF21_MEAN4
#undef EF21_MEAN
    return hipGetLastError();
}

CopyWay copy_arrays_way(const CopyList &c, int64_t state) {
    const int64_t entries = c.count[0] + c.count[1] + c.count[2];
    return copy_way(state, entries, entries == std::max(c.count[0], std::max(c.count[1], c.count[2])));
}

hipError_t launch_copy_arrays(const CopyList &c, bool streamed, hipStream_t stream) {
    const int64_t entries = c.count[0] + c.count[1] + c.count[2], per = kCopyThreads * 4;
    if (entries == 0) return hipSuccess;
    const int64_t blocks = (entries + per - 1) / per;
    const dim3 grid((unsigned)std::min<int64_t>(blocks, streamed ? 1 << 20 : kCopyBlocks)), block(kCopyThreads);
    if (streamed) hipLaunchKernelGGL(copy_arrays_kernel<true>, grid, block, 0, stream, c);
    else hipLaunchKernelGGL(copy_arrays_kernel<false>, grid, block, 0, stream, c);
    return hipGetLastError();
}

}  // namespace ef21
