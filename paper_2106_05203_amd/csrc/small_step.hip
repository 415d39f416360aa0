// One launch per iteration of Algorithm 2 for problems whose iteration is bound by launch latency rather than
// by bandwidth (dense rows, d <= 1024, a few MB of data): lines 5, 6, 8 and 3 in one kernel.
//
//   every workgroup     four row blocks of one worker's gradient (the code of the gradient kernel, so the
//                       partial sums are the same bits), then a ticket on the worker's counter;
//   the worker's last   finishes the sums to grad f_i, forms grad f_i - g_i, selects Top-k, writes the message
//   workgroup           and updates g_i (the code of the row Top-k kernel), then a ticket on the common counter;
//   the last of those   adds the messages to g in worker order and takes the model step.
//
// Where a worker's rows are few (solo_applies) ONE workgroup does all of a worker's part and no partial sums go through
// memory (solo_kernel): the gradient alone (ef21_local_grad), lines 5 and 6 with the aggregation as a second launch
// (ef21_step), or all of it in one launch with the common counter alone (EF21_ONE_LAUNCH).
//
// Nobody waits: a workgroup that is not the last to draw its ticket simply ends, so the kernel cannot hang.
// The tickets are device-scope atomics between device-scope fences (release before the ticket, acquire after
// it), which is what makes one workgroup's stores visible to another on a different compute die (draw_ticket).
#include "device_utils.h"
#include "kernels.h"
#include "logreg_dense_block.h"
#include "topk_row_impl.h"

namespace ef21 {
namespace {

constexpr int kBlocksPerWg = kRowThreads / kDenseThreads;   // 4 row blocks per workgroup of 1024 threads
constexpr int kMaxCols = 1024;                              // d of the fused iteration
constexpr int kMaxEntries = 2048;                           // n * k
// A workgroup per worker where its sixteen wavefronts have the rows in two trips (128 KB and more in flight each); with more, the
// separate kernels are ahead.  step and gradient, us, calls back to back, by the separate kernels and so: n = 4, m = 250,
// d = 100 11.9 and 8.6, 8.6 and 4.6; 4, 500, 100 11.8 and 10.4, 8.8 and 5.3; 2, 256, 256 14.1 and 13.1, 9.1 and 5.1; 30, 128, 500
// 17.9 and 17.0, 9.0 and 5.1; but step of 4, 1000, 60 10.2 and 10.3; 4, 1000, 100 12.0 and 13.0; 20, 1300, 100 13.3 and 15.5.
// And up to as many workers as there are compute units: the sums and the staged messages take most of a unit's LDS, so
// more workers take turns, where the separate kernels' workgroups lie side by side.  step, us: 256, 100, 300 33.3 and 28.3; 257, 100,
// 300 35.2 and 37.5; 257, 20, 500 33.9 and 36.0; 300, 1, 96 29.3 and 30.9; 400, 128, 500 54.6 and 54.6.
constexpr int kSoloCols = 512, kSoloTrips = 2;
constexpr int32_t kSoloWorkers = 256;
constexpr int kMaxAddSteps = 512;                           // n * ceil(k / 64), the adding wavefront's steps

struct SmallArgs {
    const float *A, *y;
    const float *x_in;        // solo_kernel: the point of the gradient, worker i's at x_in + i * x_stride
    float *x, *g, *g_i, *part, *grad;
    int32_t *msg_idx;
    float *msg_val;
    uint32_t *tickets;        // [n + 1], zero between launches
    int32_t n;
    int64_t m, d, k, rows_per_wg, chunks;
    float lambda, inv_n, neg_gamma;
    int loss, step;           // step != 0: line 3 after line 8
    const int32_t *batch;     // solo_kernel: Algorithm 5 (m rows of m_full each)
    int64_t m_full, x_stride;
};

// Line 8, then line 3, by the workgroup that drew the last ticket of all: the messages staged in LDS, ONE wavefront adds them
// worker by worker (positions inside a message are distinct, a wavefront's LDS accesses execute in program order).
struct AddShared {
    int32_t m_idx[kMaxEntries];
    float m_val[kMaxEntries];
};
__device__ __forceinline__ void add_messages(const SmallArgs &a, AddShared &sh, float *cache) {
    const int tid = threadIdx.x;
    int32_t (&m_idx)[kMaxEntries] = sh.m_idx;
    float (&m_val)[kMaxEntries] = sh.m_val;
    const int64_t total = (int64_t)a.n * a.k;
    for (int64_t t = tid; t < total; t += kRowThreads) {
        m_idx[t] = a.msg_idx[t];
        m_val[t] = a.msg_val[t];
    }
    for (int64_t j = tid; j < a.d; j += kRowThreads) cache[j] = 0.f;
    if (tid <= a.n) a.tickets[tid] = 0u;                    // n + 1 <= 1024: every ticket has been drawn
    const float gj = tid < a.d ? a.g[tid] : 0.f;            // d <= 1024: one coordinate per thread
    const float xj = a.step && tid < a.d ? a.x[tid] : 0.f;
    __syncthreads();
    if (tid < kWave) {
        for (int32_t w = 0; w < a.n; ++w) {
            for (int64_t i0 = 0; i0 < a.k; i0 += kWave) {
                const int64_t i = i0 + tid;
                if (i < a.k) cache[m_idx[w * a.k + i]] += m_val[w * a.k + i];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
    __syncthreads();
    if (tid < a.d) {
        const float gn = fmaf(cache[tid], a.inv_n, gj);
        a.g[tid] = gn;
        if (a.step) a.x[tid] = fmaf(a.neg_gamma, gn, xj);
    }
}

template <int LANES, int NQ, int SHAPE>
__global__ __launch_bounds__(kRowThreads) void small_step_kernel(SmallArgs a) {
    __shared__ RowShared s;
    __shared__ __attribute__((aligned(16))) float red[kBlocksPerWg][NQ * LANES * 4];
    __shared__ float cache[kMaxCols];
    __shared__ AddShared sh;
    __shared__ uint32_t last;
    const int tid = threadIdx.x;
    const int64_t worker = blockIdx.y;

    // ---- line 5, first half: row blocks of grad f_i
    {
        const int vb = tid / kDenseThreads;
        const int64_t chunk = (int64_t)blockIdx.x * kBlocksPerWg + vb;
        dense_block<LANES, NQ, dense_rows_in_flight<LANES, NQ, false>(), SHAPE, false>(
            a.A, a.y, a.x, a.part, a.m, a.d, a.rows_per_wg, a.loss, nullptr, a.m, worker, chunk, a.chunks,
            wave_id() % kDenseWaves, tid % kDenseThreads, chunk < a.chunks, red[vb]);
    }
    if (!draw_ticket(&a.tickets[worker], gridDim.x, &last)) return;     // the partial sums of the others, or done

    // ---- lines 5 and 6 for this worker
    {
        TopkArgs p{nullptr, a.g_i, a.n, a.d, a.k, a.msg_idx, a.msg_val, a.g_i,
                   GradParts{a.part, a.chunks, a.m, a.x, a.lambda}};
        row_topk_parts<kAddUpdate>(s, cache, p, worker);
    }
    if (!draw_ticket(&a.tickets[a.n], (uint32_t)a.n, &last)) return;      // all messages, or done

    add_messages(a, sh, cache);
}

// One workgroup per worker.  The gradient's sums stay in LDS, in fp64.  What bounds it is a chain: the worker's rows through
// one compute unit (a trip of 128 KB takes about 1.5 us), the sums over sixteen wavefronts, the selection.  Against the
// separate kernels see kSoloTrips.
enum SoloMode { kSoloGrad = 0, kSoloSelect = 1 /* lines 5 and 6 */, kSoloWhole = 2 /* lines 5, 6, 8, 3 */ };
template <int LANES, int NQ, int SHAPE, bool BATCH, int MODE>
__global__ __launch_bounds__(kRowThreads) void solo_kernel(SmallArgs a) {
    __shared__ double lds[kSoloWaves * NQ * LANES * 4];
    const int64_t worker = blockIdx.x;
    const float *x = a.x_in + worker * a.x_stride;
    if constexpr (MODE == kSoloGrad) {
        solo_gradient<LANES, NQ, SHAPE, BATCH>(a.A, a.y, x, a.m, a.d, a.lambda, a.loss, a.batch, a.m_full, worker, lds,
                                               [&](int c, float g) { a.grad[worker * a.d + c] = g; });
    } else {
        __shared__ RowShared s;
        __shared__ float cache[kSoloCols];
        const float *b = a.g_i + worker * a.d;
        const float own = (int64_t)threadIdx.x < a.d ? b[threadIdx.x] : 0.f;      // fetched beside the rows
        solo_gradient<LANES, NQ, SHAPE, BATCH>(a.A, a.y, x, a.m, a.d, a.lambda, a.loss, a.batch, a.m_full, worker, lds,
                                               [&](int c, float g) { cache[c] = g - own; });
        __syncthreads();
        const TopkArgs p{nullptr, a.g_i, a.n, a.d, a.k, a.msg_idx, a.msg_val, a.g_i};
        row_topk_on<kAddUpdate>(
            s, p, worker, [&](int64_t e) { return cache[e]; }, [&](int64_t e) { return b[e]; });
        if constexpr (MODE == kSoloWhole) {
            __shared__ AddShared sh;
            __shared__ uint32_t last;
            if (!draw_ticket(&a.tickets[a.n], (uint32_t)a.n, &last)) return;
            add_messages(a, sh, cache);
        }
    }
}

template <int LANES, int NQ>
void launch(const SmallArgs &a, hipStream_t stream) {
    const dim3 grid((unsigned)((a.chunks + kBlocksPerWg - 1) / kBlocksPerWg), (unsigned)a.n);
    const dim3 block(kRowThreads);
    if (a.d % 4 == 0) hipLaunchKernelGGL((small_step_kernel<LANES, NQ, kQuadRows>), grid, block, 0, stream, a);
    else if (a.d > 4) hipLaunchKernelGGL((small_step_kernel<LANES, NQ, kRaggedRows>), grid, block, 0, stream, a);
    else if constexpr (LANES == 16) hipLaunchKernelGGL((small_step_kernel<LANES, NQ, kTinyRows>), grid, block, 0, stream, a);
}

}  // namespace

namespace {
template <int LANES, int NQ, int SHAPE, int MODE>
void launch_solo_shape(const SmallArgs &a, hipStream_t stream) {
    const dim3 grid((unsigned)a.n), block(kRowThreads);
    if constexpr (MODE != kSoloWhole) {
        if (a.batch) {
            hipLaunchKernelGGL((solo_kernel<LANES, NQ, SHAPE, true, MODE>), grid, block, 0, stream, a);
            return;
        }
    }
    hipLaunchKernelGGL((solo_kernel<LANES, NQ, SHAPE, false, MODE>), grid, block, 0, stream, a);
}

template <int MODE>
hipError_t launch_solo(const SmallArgs &a, hipStream_t stream) {
    const bool quads = a.d % 4 == 0;
    const DenseVariant dv = dense_variant(a.d);
#define EF21_SOLO(LANES, NQ)                                                                      \
    do {                                                                                          \
        if (quads) launch_solo_shape<LANES, NQ, kQuadRows, MODE>(a, stream);                      \
        else launch_solo_shape<LANES, NQ, kRaggedRows, MODE>(a, stream);                          \
    } while (0)
    switch (dv.lanes * 100 + dv.nq) {
        case 1601:
            if (a.d < 4) launch_solo_shape<16, 1, kTinyRows, MODE>(a, stream);
            else EF21_SOLO(16, 1);
            break;
        case 3201: EF21_SOLO(32, 1); break;
        case 6401: EF21_SOLO(64, 1); break;
        case 6402: EF21_SOLO(64, 2); break;
        default: return hipErrorInvalidValue;
    }
#undef EF21_SOLO
    return hipGetLastError();
}
}  // namespace

bool solo_applies(int32_t n, int64_t m, int64_t m_full, int64_t d) {
    const int64_t trip = dense_trip_rows(d, false) * (kSoloWaves / kDenseWaves);
    return n <= kSoloWorkers && d <= kSoloCols && m <= kSoloTrips * trip && !dense_deep(n, m_full, d);
}

hipError_t launch_solo_grad(const float *A, const float *y, const float *x, float *grad, int32_t n, int64_t m_full,
                            int64_t d, float lambda, int loss, RowBatch rb, int64_t x_stride, hipStream_t stream) {
    SmallArgs a{};
    a.A = A;
    a.y = y;
    a.x_in = x;
    a.grad = grad;
    a.n = n;
    a.m = rb.tau > 0 ? rb.tau : m_full;
    a.d = d;
    a.lambda = lambda;
    a.loss = loss;
    a.batch = rb.tau > 0 ? rb.rows : nullptr;
    a.m_full = m_full;
    a.x_stride = x_stride;
    if (!solo_applies(n, a.m, m_full, d)) return hipErrorInvalidValue;
    return launch_solo<kSoloGrad>(a, stream);
}

hipError_t launch_solo_select(const float *A, const float *y, const float *x, float *g_i, int32_t n, int64_t m_full, int64_t d,
                              int64_t k, float lambda, int loss, RowBatch rb, int32_t *msg_idx, float *msg_val,
                              hipStream_t stream) {
    SmallArgs a{};
    a.A = A;
    a.y = y;
    a.x_in = x;
    a.g_i = g_i;
    a.msg_idx = msg_idx;
    a.msg_val = msg_val;
    a.n = n;
    a.m = rb.tau > 0 ? rb.tau : m_full;
    a.d = d;
    a.k = k;
    a.lambda = lambda;
    a.loss = loss;
    a.batch = rb.tau > 0 ? rb.rows : nullptr;
    a.m_full = m_full;
    if (!solo_applies(n, a.m, m_full, d)) return hipErrorInvalidValue;
    return launch_solo<kSoloSelect>(a, stream);
}

bool small_step_applies(int32_t n, int64_t m, int64_t d, int64_t k) {
    return d <= kMaxCols && dense_variant(d).lanes != 0 && n < kRowThreads && (int64_t)n * k <= kMaxEntries &&
           (int64_t)n * ((k + kWave - 1) / kWave) <= kMaxAddSteps && (int64_t)n * m * d <= kSmallProblem;
}

size_t small_step_ticket_bytes(int32_t n) { return sizeof(uint32_t) * ((size_t)n + 1); }

hipError_t launch_small_step(const float *A, const float *y, float *x, float *g, float *g_i, int32_t n, int64_t m,
                             int64_t d, int64_t k, float lambda, float gamma, int loss, bool take_step, void *scratch,
                             void *tickets, int32_t *msg_idx, float *msg_val, hipStream_t stream) {
    if (!small_step_applies(n, m, d, k)) return hipErrorInvalidValue;
    const DensePlan pl = dense_plan(n, m, d, false);
    SmallArgs a{};
    a.A = A;
    a.y = y;
    a.x_in = x;
    a.x = x;
    a.g = g;
    a.g_i = g_i;
    a.part = (float *)scratch;
    a.msg_idx = msg_idx;
    a.msg_val = msg_val;
    a.tickets = (uint32_t *)tickets;
    a.n = n;
    a.m = a.m_full = m;
    a.d = d;
    a.k = k;
    a.rows_per_wg = pl.rows_per_wg;
    a.chunks = pl.chunks;
    a.lambda = lambda;
    a.inv_n = 1.0f / (float)n;
    a.neg_gamma = -gamma;
    a.loss = loss;
    a.step = take_step ? 1 : 0;
    if (solo_applies(n, m, m, d)) return launch_solo<kSoloWhole>(a, stream);
    const DenseVariant dv = dense_variant(d);
    switch (dv.lanes * 100 + dv.nq) {
        case 1601: launch<16, 1>(a, stream); break;
        case 3201: launch<32, 1>(a, stream); break;
        case 6401: launch<64, 1>(a, stream); break;
        case 6402: launch<64, 2>(a, stream); break;
        case 6404: launch<64, 4>(a, stream); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace ef21
