// Host-side launchers of the HIP kernels.  Each enqueues on `stream` and returns the HIP status
// of the launch; none of them allocates or synchronises.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "copy_way.h"

namespace ef21 {

// Runs `setup` once per HIP device, with that device current: for attributes of a kernel (such as its dynamic LDS
// limit), which the runtime keeps per device.  Thread-safe; a failed setup is tried again by the next call.
struct PerDeviceOnce {
    std::mutex mu;
    bool done[64] = {};
    template <class Setup>
    hipError_t operator()(Setup setup) {
        int dev = 0;
        hipError_t st = hipGetDevice(&dev);
        if (st != hipSuccess) return st;
        if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
        std::lock_guard<std::mutex> lock(mu);
        if (done[dev]) return hipSuccess;
        st = setup();
        if (st == hipSuccess) done[dev] = true;
        return st;
    }
};

// Kernel classes for the optional per-kernel timing of a handle (EF21_K_* in include/ef21.h).
enum KernelId {
    K_GRAD_MAIN = 0,   // the pass(es) over the problem data
    K_GRAD_AUX,        // partial-sum reduction / regulariser
    K_TOPK_ROW,        // one-workgroup-per-row Top-k (+ fused update)
    K_TOPK_COLLECT,    // long rows: the pass over the row that collects candidates
    K_TOPK_SELECT,     // long rows, k = 1: the message of the running maximum (+ fused update)
    K_TOPK_REFINE,     // no kernel: callers' arrays are laid out by these numbers
    K_TOPK_COUNT,      // long rows, large k: per-slot counts
    K_TOPK_EMIT,       // long rows, large k: ordered emission (+ fused update)
    K_MODEL_STEP,      // g <- g + mean of the messages and / or x <- x - gamma g
    K_PLUS,            // Algorithm 3: distortions, choice and update of g_i, mean of the rows
    K_SMALL_STEP,      // the whole iteration of Algorithm 2 in one launch (small dense problems)
    K_COUNT
};

// Called after each kernel launch with the class of the kernel just enqueued; a default-constructed
// Marker does nothing.
struct Marker {
    void (*fn)(void *user, int kernel_id) = nullptr;
    void *user = nullptr;
    void operator()(int kernel_id) const {
        if (fn) fn(user, kernel_id);
    }
};

// A dense gradient of eq. (9) left as per-row-block partial sums part[n][chunks][d]: entry (i, j) is
// dense_grad_entry(part + i * chunks * d, chunks, d, j, x[j], m, lambda) (logreg_finish.h).
struct GradParts {
    const float *part = nullptr;
    int64_t chunks = 0;
    int64_t m = 0;
    const float *x = nullptr;
    float lambda = 0.f;
};

// Arguments of one batched Top-k (Section 2.1) over n rows of length d.
//   a, b      v = a - b if b != nullptr (the difference of Algorithm 2, line 5), else v = a
//   out_idx, out_val   [n][k] ascending positions and signed values
//   g_i       if != nullptr the kept entries also update the workers' state in place:
//             b != nullptr (then g_i is the same array): g_i[row][j] = b[row][j] + v (Algorithm 2, line 6)
//             b == nullptr (then g_i is the same array as a): g_i[row][j] = 0 (Algorithm 4, e_i = p_i - w_i)
struct TopkArgs {
    const float *a;
    const float *b;
    int32_t n;
    int64_t d;
    int64_t k;
    int32_t *out_idx;
    float *out_val;
    float *g_i;
    GradParts parts;   // if parts.part != nullptr the rows of `a` are these unreduced gradients (`a` is not read);
                       // launch_topk_row only, d <= kRowPartsMax, b != nullptr
    int32_t warm;      // launch_topk_split only, k >= 2: 0, or 1 = the row thresholds of the last such call on this
                       // workspace serve as the first guess of this call's (the result never depends on it; meant
                       // for consecutive iterations of one algorithm on one state)
    // launch_topk_split with k > 1 and launch_topk_row_reg only: if agg_start != nullptr the emission also writes the index that
    // launch_aggregate needs of the messages (aggregate_index_shift), so that its own indexing kernel can be skipped
    int32_t *agg_start;
    int32_t agg_shift;
    int64_t agg_nblk;
    // launch_topk_split with warm = 1, k >= 2, b == nullptr and g_i == a only: if add != nullptr the rows are
    // a + add_scale * add (one fused multiply-add per entry), written over a by the pass that reads them
    const float *add;
    float add_scale;
};

// Rows this long can be handed to launch_topk_row as unreduced gradients (TopkArgs::parts).
constexpr int64_t kRowPartsMax = 4096;
// Up to this length they are (launch_logreg_grad_dense).  Longer ones are finished by a kernel that the whole chip shares, and
// launch_topk_row_reg selects from the differences.  step, us, unreduced and finished, k = d / 20: d = 700: n = 10, m = 8 16.1
// and 16.7, n = 32, m = 500 23.5 and 24.2, n = 10, m = 2000 24.0 and 23.7; d = 900: n = 4, m = 500 18.3 and 17.8, n = 10, m = 2000 28.0
// and 26.9; d = 1200: 21.6 and 19.7, 35.0 and 32.4; d = 2000: 26.0 and 20.8, 48.5 and 43.7.
constexpr int64_t kRowPartsCols = 900;
// With up to kRowPartsFew sums per column, unreduced costs the Top-k kernel next to nothing and saves a launch: up to this length
// against the selection from registers (m = 8, the same way: n = 4, d = 900 15.7 and 16.2; d = 1000 15.8 and 16.4; n = 10 17.3 and 17.4;
// n = 4, d = 1200 17.7 and 17.8; d = 1500 19.1 and 18.5), and up to kRowPartsMax where too many entries are kept for that one and
// both select from LDS (k = d / 5: n = 1, m = 8, d = 950 15.2 and 17.0; n = 4, m = 32, d = 1507 21.5 and 22.7; n = 32, m = 16, d = 2500 26.5
// and 27.6; n = 1, m = 2, d = 4000 24.6 and 25.0; eight sums: n = 1, m = 64, d = 1507 21.3 and 20.9, d = 2500 26.2 and 24.4).
constexpr int64_t kRowPartsFew = 4, kRowPartsFewCols = 1200;

// One workgroup per row: a histogram pass over the row and a ranking of the threshold's bin (three histogram passes where
// the bin is crowded), then an ordered emission.  Needs no workspace; rows of at most 16384 entries.
hipError_t launch_topk_row(const TopkArgs &p, hipStream_t stream);

// One workgroup per row that keeps the row in registers: rows of kRowRegMin to kRowRegMax entries, given as they are or as
// a difference, k <= kRowRegMaxK.  No workspace.  Other shapes: hipErrorInvalidValue.
constexpr int64_t kRowRegMin = 512, kRowRegMax = 61440, kRowRegMaxK = 1024;
hipError_t launch_topk_row_reg(const TopkArgs &p, hipStream_t stream);

// Many workgroups per row for long rows.  Workspace layout and size: topk_split_workspace_bytes.
size_t topk_split_workspace_bytes(int32_t n, int64_t d, int64_t k);
hipError_t launch_topk_split(const TopkArgs &p, void *workspace, hipStream_t stream, const Marker &mk = Marker());
// Two selections of one pass over the same arrays (Algorithm 3, lines 5 to 7): `plain` selects from the rows of a,
// `markov` from a - b (plain.a == markov.a, plain.b == nullptr, same n, d, k >= 2, no g_i update, warm both or
// neither), each with a workspace of its own.  The sums of line 7 come along, all in fp64 in a fixed order, per row and
// per piece of the row (topk_split_slots(n, d) pieces):
struct PairSums {
    void *norms;              // double2 [n][slots]: (sum a^2, sum (a - b)^2), differences taken exactly
    double *kept_plain;       // [n][slots]: the kept entries of a, squared
    double *kept_markov;      // [n][slots]: the kept entries of a - b, unrounded, squared
    float *resid;             // scratch [n][topk_split_slot_entries(n, d)]; nullptr: a and b are read again (slower)
};
int64_t topk_split_slots(int32_t n, int64_t d);
int64_t topk_split_slot_entries(int32_t n, int64_t d);       // candidates of a row that its slots have room for
hipError_t launch_topk_split_pair(const TopkArgs &plain, const TopkArgs &markov, void *ws_plain, void *ws_markov,
                                  const PairSums &sums, hipStream_t stream, const Marker &mk = Marker());
// The kernels keep the workspace's histograms and tickets zeroed as long as (n, d) stay the same.
// A workspace that is new, or was last used with another (n, d), needs this reset first.
hipError_t launch_topk_split_reset(void *workspace, int32_t n, int64_t d, hipStream_t stream);

// Algorithm 2, line 3: x <- x - gamma g.
hipError_t launch_model_step(float *x, const float *g, int64_t d, float gamma, hipStream_t stream);

// Algorithm 2, line 8: g <- g + (1/n) sum_i c_i from the messages (idx, val) [n][k] (positions ascending
// and distinct inside a row), summed without global atomics in an order that n, d and k alone fix: the workers' own, except
// with many workers (kManyWorkers in update.hip) on more than small messages, where four runs of consecutive workers are
// summed side by side; if x != nullptr followed, in the same pass over the coordinates, by line 3 with the new g.
// `index`: aggregate_index_bytes(n, d) bytes of scratch, overwritten by every call.
// The index: start[w][b] = first pair of worker w's message at or beyond coordinate b << shift, for the blocks
// b = 0 .. nblk of 2^shift coordinates (start[w][nblk] = k), int32 [n][nblk + 1].  aggregate_index_shift gives the
// shift that launch_aggregate uses for a shape (nblk = ceil(d / 2^shift)), or -1 if it uses no index for it.
// index_ready: the caller has already written the index (launch_topk_split can); otherwise a kernel of the call does.
size_t aggregate_index_bytes(int32_t n, int64_t d);
int aggregate_index_shift(int32_t n, int64_t k, int64_t d);
// from_zero: g is not read, (1/n) sum_i c_i is written.
hipError_t launch_aggregate(const int32_t *idx, const float *val, int32_t n, int64_t k, int64_t d, float *g, float *x,
                            float gamma, void *index, hipStream_t stream, bool index_ready = false,
                            bool from_zero = false);

// g = (1/n) sum_i g_i (input line of Algorithm 2), summed in worker order; in the same launch, if rows_out != nullptr, rows_out <-
// g_i and, if x_out != nullptr as well, x_out [d] <- x (a caller does not ask for copies where mean_way says kMemcpy).
hipError_t launch_mean_rows(const float *g_i, float *g, int32_t n, int64_t d, hipStream_t stream, float *rows_out = nullptr,
                            const float *x = nullptr, float *x_out = nullptr);

// dst[a][0 .. count[a]) <- src[a] for up to three arrays (count 0: none) in one launch.
struct CopyList {
    const float *src[3];
    float *dst[3];
    int64_t count[3];
};
CopyWay copy_arrays_way(const CopyList &c, int64_t state);       // state: see copy_way
hipError_t launch_copy_arrays(const CopyList &c, bool streamed, hipStream_t stream);

// `loss` below: the per-row loss of the linear model (LossKind in device_utils.h): logistic (eq. (9)) or squared.
// kLossHalfSquare (z^2 / 2, no target) is internal: its gradient is (1/m) A_i^T A_i x, the product the power
// iteration needs.  x_stride below: 0 = one x [d] for all workers, d = a row of x [n][d] per worker.
enum { kLossLogistic = 0, kLossLeastSquares = 1, kLossHalfSquare = 2 };

// The minibatch of Algorithm 5: worker i's gradient estimator sums the rows rows[i][0..tau) of its m rows
// (tau <= m; an entry outside [0, m) contributes nothing) and divides by tau.  tau == 0: all rows, the gradient.
struct RowBatch {
    const int32_t *rows = nullptr;   // device, [n][tau]
    int64_t tau = 0;
};

// Gradient of eq. (9) for all workers, dense rows.  scratch: logreg_dense_scratch_bytes.  With defer != nullptr
// the last reduction may be left to the consumer: then *defer describes the partial sums (they live in
// scratch until the next call) and grad is not written; defer->part == nullptr means grad was written.  few_cols: the most columns
// of which it leaves a few sums (kRowPartsFewCols or kRowPartsMax).
size_t logreg_dense_scratch_bytes(int32_t n, int64_t m, int64_t d);
hipError_t launch_logreg_grad_dense(const float *A, const float *y, const float *x, float *grad, int32_t n,
                                    int64_t m, int64_t d, float lambda, void *scratch, hipStream_t stream,
                                    const Marker &mk = Marker(), GradParts *defer = nullptr,
                                    int loss = kLossLogistic, RowBatch batch = RowBatch(), int64_t x_stride = 0,
                                    int64_t few_cols = kRowPartsFewCols);

// Gradient of eq. (9) for all workers, CSR rows with nnz entries in all.  `index`
// (logreg_csr_index_bytes bytes, owned by the caller) is built once per problem by logreg_csr_build_index
// and holds per-row column-range offsets, a range-major and a column-major copy of the matrix (6 bytes per
// entry each) and scratch for the two-pass kernels.  The build synchronises the stream and reports whether those
// kernels can be used (every row's columns ascending and inside [0, d), fewer than 2^31 entries per
// worker); pass index = nullptr to launch_logreg_grad_csr otherwise.  Under a row batch the work is
// proportional to the batch: one wavefront per listed row and global fp32 atomics, whatever the index.
size_t logreg_csr_index_bytes(int32_t n, int64_t m, int64_t d, int64_t nnz);
hipError_t logreg_csr_build_index(const int64_t *rowptr, const int32_t *col, const float *val, int32_t n, int64_t m,
                                  int64_t d, int64_t nnz, void *index, hipStream_t stream, bool *usable);
hipError_t launch_logreg_grad_csr(const int64_t *rowptr, const int32_t *col, const float *val, const float *y,
                                  const float *x, float *grad, int32_t n, int64_t m, int64_t d, int64_t nnz,
                                  float lambda, const void *index, hipStream_t stream, const Marker &mk = Marker(),
                                  int loss = kLossLogistic, RowBatch batch = RowBatch(), int64_t x_stride = 0);

// Dense problems with few rows per worker (m of m_full, d columns), a workgroup per worker: the gradient, or lines 5 and 6 of
// Algorithm 2 (the messages, and g_i updated in place).  The gradient's bits are the same either way.  launch_logreg_grad_dense
// takes the first by itself.
bool solo_applies(int32_t n, int64_t m, int64_t m_full, int64_t d);
hipError_t launch_solo_grad(const float *A, const float *y, const float *x, float *grad, int32_t n, int64_t m_full,
                            int64_t d, float lambda, int loss, RowBatch batch, int64_t x_stride, hipStream_t stream);
hipError_t launch_solo_select(const float *A, const float *y, const float *x, float *g_i, int32_t n, int64_t m_full,
                              int64_t d, int64_t k, float lambda, int loss, RowBatch batch, int32_t *msg_idx,
                              float *msg_val, hipStream_t stream);

// Small dense problems: lines 5, 6, 8 (and 3 if take_step) of Algorithm 2 in ONE launch, from the problem and the
// state, with the arithmetic of the separate kernels (gradient, row Top-k with update, aggregation), so the
// results are the same bits.  small_step_applies says whether the shape qualifies (d <= 1024, n * k <= 2048,
// n * m * d <= 2^24, ...).  scratch: logreg_dense_scratch_bytes; tickets: small_step_ticket_bytes(n) bytes,
// zero before the first launch (the kernel leaves them zero).
bool small_step_applies(int32_t n, int64_t m, int64_t d, int64_t k);
size_t small_step_ticket_bytes(int32_t n);
hipError_t launch_small_step(const float *A, const float *y, float *x, float *g, float *g_i, int32_t n, int64_t m,
                             int64_t d, int64_t k, float lambda, float gamma, int loss, bool take_step, void *scratch,
                             void *tickets, int32_t *msg_idx, float *msg_val, hipStream_t stream);

// Algorithm 3 (EF21+), lines 7 and 8, for all workers: from the gradients s [n][d], the estimators g_i [n][d]
// (updated in place) and the two Top-k results (idx_b, val_b) = C(s), (idx_m, val_m) = C(s - g_i), all [n][k]:
// BM[i] = (B_i, M_i), branch[i] = 1 where the plain compressor wins (M_i > B_i), (msg_idx, msg_val) = the chosen
// pairs, and g_i <- b or m accordingly.  scratch: plus_scratch_bytes(n, d, k) bytes.
size_t plus_scratch_bytes(int32_t n, int64_t d, int64_t k);
hipError_t launch_plus_choose(const float *s, float *g_i, int32_t n, int64_t d, int64_t k, const int32_t *idx_b,
                              const float *val_b, const int32_t *idx_m, const float *val_m, void *scratch,
                              int32_t *branch, double *BM, int32_t *msg_idx, float *msg_val, hipStream_t stream);

// The same for long rows, with line 10 (g = mean of the rows) and, if x != nullptr, the model step, after
// launch_topk_split_pair has left the two selections, their message indexes (blocks of 2^kPlusShift coordinates) and
// the sums of line 7 in what plus_long_layout describes (it returns the bytes; scratch may be nullptr).
constexpr int kPlusShift = 9;
struct PlusLong {
    void *norms;                          // PairSums
    double *kept_plain, *kept_markov;
    int32_t *start_plain, *start_markov;  // TopkArgs::agg_start
    int64_t nblk;
};
struct PlusLongArgs {
    int32_t n;
    int64_t d, k;
    const int32_t *idx_b, *idx_m;         // the two selections, [n][k]
    const float *val_b, *val_m;
    float *g_i, *g, *x;
    int32_t *branch, *msg_idx;
    float *msg_val;
    const int32_t *start_b, *start_m;     // filled in by launch_plus_long
    int64_t nblk;
};
size_t plus_long_layout(int32_t n, int64_t d, void *scratch, PlusLong *out);
hipError_t launch_plus_long(const PlusLong &pl, PlusLongArgs a, double *BM, float gamma, hipStream_t stream);

// Power iteration for the smoothness constants of Section 3.4: v [rows][d] <- a fixed positive start vector;
// and one step: stats[row] = (v^T w / v^T v, |w| / |v|) as two doubles, v <- w / |w|, for w = M v, M symmetric
// positive semidefinite (both numbers are lower bounds of its largest eigenvalue).
hipError_t launch_power_start(float *v, int32_t rows, int64_t d, hipStream_t stream);
hipError_t launch_power_step(const float *w, float *v, int32_t rows, int64_t d, double *stats, hipStream_t stream);

// The same on the Gram matrices of a dense problem (d <= 1024), a workspace of gram_way's bytes and its squarings (gram_way.h).
// stats [n + 1] pairs as above, the last one of the whole problem; the first number of a pair is not formed (0).
hipError_t launch_gram_power(const float *A, int32_t n, int64_t m, int64_t d, int32_t iterations, int32_t squarings, void *workspace,
                             double *stats, hipStream_t stream);

// Algorithm 4 (EF): e <- e + gamma s over all n * d entries.
hipError_t launch_ef_accumulate(const float *s, float *e, int32_t n, int64_t d, float gamma, hipStream_t stream);

// Plain streaming kernels for measuring what the HBM delivers: one read of `n16` 16-byte words (their sum goes
// to sink[0]), and a copy.
hipError_t launch_hbm_read(const void *src, int64_t n16, float *sink, hipStream_t stream);
hipError_t launch_hbm_copy(void *dst, const void *src, int64_t n16, hipStream_t stream);

}  // namespace ef21
