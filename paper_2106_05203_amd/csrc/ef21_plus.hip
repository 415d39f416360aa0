// EF21+ (Algorithm 3 of the EF21 paper): per worker, the better of the plain compressor b = C(s) and the
// Markov compressor m = g_i + C(s - g_i), s = grad f_i(x), C = Top-k.  The two Top-k selections are the
// library's ordinary ones; this file holds what is particular to Algorithm 3:
//   line 7  the distortions B = ||b - s||^2 = ||s||^2 - sum of the kept s_j^2 and
//           M = ||m - s||^2 = ||s - g_i||^2 - sum of the kept (s_j - g_ij)^2 (at a kept position m_j equals s_j
//           up to the rounding of one fp32 addition), differences and sums in fp64, in a fixed order;
//   line 8  g_i <- m if M <= B, else b: a sparse update, or a rewrite of the whole row;
//   line 10 g = (1/n) sum_i g_i is then recomputed from the rows (launch_mean_rows).
// Long rows (launch_plus_long): the norms and the kept sums come from the kernels of the two selections, and lines 8, 10
// and the model step are one pass over the coordinates.
#include "device_utils.h"
#include "kernels.h"

namespace ef21 {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int64_t kNormChunk = 1 << 16;      // entries of a row per workgroup of the norm / rewrite kernels

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// Sum over the workgroup, the same value in every thread; `lds` holds kWaves doubles.
__device__ double block_sum_f64(double v, double *lds) {
    v = wave_sum_f64(v);
    __syncthreads();                       // lds may still be read from a previous call
    if (lane_id() == 0) lds[threadIdx.x / kWave] = v;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < kWaves; ++w) t += lds[w];
    return t;
}

// part[row][chunk] = (sum s^2, sum (s - g_i)^2) over the chunk, the differences of the stored values taken
// exactly (in fp64), as the distortions of line 7 are defined on the stored vectors.  VEC = 4 (rows of a
// multiple of four entries, 16-byte aligned): four float4 loads per array in flight per thread.
template <int VEC>
__global__ __launch_bounds__(kThreads) void plus_sqnorms_kernel(const float *__restrict__ s,
                                                                const float *__restrict__ g_i, int64_t d,
                                                                double2 *__restrict__ part) {
    __shared__ double lds[kWaves];
    const int64_t row = blockIdx.y, chunk = blockIdx.x;
    const int64_t lo = chunk * kNormChunk, hi = lo + kNormChunk < d ? lo + kNormChunk : d;
    const float *sr = s + row * d, *gr = g_i + row * d;
    double acc_s = 0.0, acc_v = 0.0;
    if constexpr (VEC == 4) {
        constexpr int kUnroll = 4;
        constexpr int64_t kStep = (int64_t)kThreads * 4;
        int64_t e = lo + (int64_t)threadIdx.x * 4;
        for (; e + (kUnroll - 1) * kStep + 4 <= hi; e += kUnroll * kStep) {
            float4 a[kUnroll], b[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                a[u] = stream_load4(sr + e + u * kStep);
                b[u] = stream_load4(gr + e + u * kStep);
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const double s0 = a[u].x, s1 = a[u].y, s2 = a[u].z, s3 = a[u].w;
                const double v0 = s0 - (double)b[u].x, v1 = s1 - (double)b[u].y, v2 = s2 - (double)b[u].z,
                             v3 = s3 - (double)b[u].w;                       // exact
                acc_s += (s0 * s0 + s1 * s1) + (s2 * s2 + s3 * s3);
                acc_v += (v0 * v0 + v1 * v1) + (v2 * v2 + v3 * v3);
            }
        }
        for (; e + 4 <= hi; e += kStep) {
            const float4 a = stream_load4(sr + e), b = stream_load4(gr + e);
            const double s0 = a.x, s1 = a.y, s2 = a.z, s3 = a.w;
            const double v0 = s0 - (double)b.x, v1 = s1 - (double)b.y, v2 = s2 - (double)b.z, v3 = s3 - (double)b.w;
            acc_s += (s0 * s0 + s1 * s1) + (s2 * s2 + s3 * s3);
            acc_v += (v0 * v0 + v1 * v1) + (v2 * v2 + v3 * v3);
        }
    } else {
        for (int64_t e = lo + threadIdx.x; e < hi; e += kThreads) {
            const double sv = (double)stream_load(sr + e), v = sv - (double)stream_load(gr + e);   // exact
            acc_s += sv * sv;
            acc_v += v * v;
        }
    }
    acc_s = block_sum_f64(acc_s, lds);
    acc_v = block_sum_f64(acc_v, lds);
    if (threadIdx.x == 0) part[row * gridDim.x + chunk] = make_double2(acc_s, acc_v);
}

// What the kept entries take away from the two norms, per block of kKeptBlock message entries:
// kept[row][blk] = (sum of b_j^2, sum of (s_j - g_ij)^2 over the positions of m).  b_j = s_j exactly; m_j = s_j
// up to the rounding of the fp32 update, so the exact (s_j - g_ij)^2 leaves the sum.
constexpr int64_t kKeptBlock = (int64_t)kThreads * 8;

__global__ __launch_bounds__(kThreads) void plus_kept_kernel(const float *__restrict__ s,
                                                             const float *__restrict__ g_i, int64_t d,
                                                             const float *__restrict__ val_b,
                                                             const int32_t *__restrict__ idx_m, int64_t k,
                                                             double2 *__restrict__ kept) {
    __shared__ double lds[kWaves];
    const int64_t row = blockIdx.y;
    const int64_t lo = (int64_t)blockIdx.x * kKeptBlock, hi = lo + kKeptBlock < k ? lo + kKeptBlock : k;
    double kb = 0.0, km = 0.0;
    for (int64_t j = lo + threadIdx.x; j < hi; j += kThreads) {
        const double vb = (double)val_b[row * k + j];
        const int64_t e = idx_m[row * k + j];
        const double vm = (double)s[row * d + e] - (double)g_i[row * d + e];
        kb += vb * vb;
        km += vm * vm;
    }
    kb = block_sum_f64(kb, lds);
    km = block_sum_f64(km, lds);
    if (threadIdx.x == 0) kept[row * gridDim.x + blockIdx.x] = make_double2(kb, km);
}

// One workgroup per worker: B, M and the choice of line 8 from the partial sums (each added in a fixed order).
// kblocks == 0 (short messages): the kept sums are taken here, from the messages themselves.
__global__ __launch_bounds__(kThreads) void plus_decide_kernel(const double2 *__restrict__ part, int64_t chunks,
                                                               const double2 *__restrict__ kept, int64_t kblocks,
                                                               const float *__restrict__ s,
                                                               const float *__restrict__ g_i, int64_t d,
                                                               const float *__restrict__ val_b,
                                                               const int32_t *__restrict__ idx_m, int64_t k,
                                                               int32_t *__restrict__ branch, double *__restrict__ BM) {
    __shared__ double lds[kWaves];
    const int64_t row = blockIdx.x;
    double ns = 0.0, nv = 0.0, kb = 0.0, km = 0.0;
    for (int64_t c = threadIdx.x; c < chunks; c += kThreads) {
        const double2 p = part[row * chunks + c];
        ns += p.x;
        nv += p.y;
    }
    for (int64_t c = threadIdx.x; c < kblocks; c += kThreads) {
        const double2 p = kept[row * kblocks + c];
        kb += p.x;
        km += p.y;
    }
    if (kblocks == 0) {
        for (int64_t j = threadIdx.x; j < k; j += kThreads) {
            const double vb = (double)val_b[row * k + j];
            const int64_t e = idx_m[row * k + j];
            const double vm = (double)s[row * d + e] - (double)g_i[row * d + e];
            kb += vb * vb;
            km += vm * vm;
        }
    }
    ns = block_sum_f64(ns, lds);
    nv = block_sum_f64(nv, lds);
    kb = block_sum_f64(kb, lds);
    km = block_sum_f64(km, lds);
    const double B = ns - kb, M = nv - km;
    if (threadIdx.x == 0) {
        branch[row] = M > B ? 1 : 0;                // line 8: the Markov compressor unless it is strictly worse
        BM[2 * row] = B;
        BM[2 * row + 1] = M;
    }
}

// Rows whose worker chose the plain compressor are cleared (g_i <- b has k non-zeros at most).
template <int VEC>
__global__ __launch_bounds__(kThreads) void plus_clear_kernel(const int32_t *__restrict__ branch,
                                                              float *__restrict__ g_i, int64_t d) {
    const int64_t row = blockIdx.y;
    if (!branch[row]) return;
    const int64_t lo = (int64_t)blockIdx.x * kNormChunk, hi = lo + kNormChunk < d ? lo + kNormChunk : d;
    float *gr = g_i + row * d;
    if constexpr (VEC == 4) {
        for (int64_t e = lo + (int64_t)threadIdx.x * 4; e + 4 <= hi; e += (int64_t)kThreads * 4)
            *reinterpret_cast<float4 *>(gr + e) = make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
        for (int64_t e = lo + threadIdx.x; e < hi; e += kThreads) gr[e] = 0.f;
    }
}

// The k entries of the chosen message, copied to (msg_idx, msg_val) and applied: added to g_i (Markov branch,
// one fp32 addition each) or written into the cleared row (plain branch).
__global__ __launch_bounds__(kThreads) void plus_apply_kernel(const int32_t *__restrict__ branch,
                                                              const int32_t *__restrict__ idx_b,
                                                              const float *__restrict__ val_b,
                                                              const int32_t *__restrict__ idx_m,
                                                              const float *__restrict__ val_m, int64_t k,
                                                              int32_t *__restrict__ msg_idx,
                                                              float *__restrict__ msg_val, float *__restrict__ g_i,
                                                              int64_t d) {
    const int64_t row = blockIdx.y;
    const bool plain = branch[row] != 0;
    const int32_t *ci = plain ? idx_b : idx_m;
    const float *cv = plain ? val_b : val_m;
    float *gr = g_i + row * d;
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    for (int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x; j < k; j += stride) {
        const int32_t e = ci[row * k + j];
        const float v = cv[row * k + j];
        msg_idx[row * k + j] = e;
        msg_val[row * k + j] = v;
        gr[e] = plain ? v : gr[e] + v;
    }
}

// ---- long rows
// One workgroup per worker: B, M and the choice of line 8 from the sums per piece of the row.
__global__ __launch_bounds__(kThreads) void plus_decide_long_kernel(const double2 *__restrict__ norms,
                                                                    const double *__restrict__ kept_b,
                                                                    const double *__restrict__ kept_m, int64_t slots,
                                                                    int32_t *__restrict__ branch,
                                                                    double *__restrict__ BM) {
    __shared__ double lds[kWaves];
    const int64_t row = blockIdx.x;
    double ns = 0.0, nv = 0.0, kb = 0.0, km = 0.0;
    for (int64_t c = threadIdx.x; c < slots; c += kThreads) {
        const double2 p = norms[row * slots + c];
        ns += p.x;
        nv += p.y;
        kb += kept_b[row * slots + c];
        km += kept_m[row * slots + c];
    }
    ns = block_sum_f64(ns, lds);
    nv = block_sum_f64(nv, lds);
    kb = block_sum_f64(kb, lds);
    km = block_sum_f64(km, lds);
    if (threadIdx.x == 0) {
        const double B = ns - kb, M = nv - km;
        branch[row] = M > B ? 1 : 0;                // line 8: the Markov compressor unless it is strictly worse
        BM[2 * row] = B;
        BM[2 * row + 1] = M;
    }
}

// Lines 8 and 10, and with STEP line 3, for a block of kApplyCols coordinates per wavefront: worker after worker, the
// row's old values (Markov branch; zeros otherwise) go to LDS, the run of the chosen message inside the block is added
// to them or written over them, and the new values are added to the sum in fp64.  A Markov row changes at the run's
// positions only and is written there; a row that switches to the plain compressor is written whole.  The chosen pairs
// are copied to the message buffers on the way.  What bounds it: the rows' bytes, read once and, where replaced,
// written once (n = 5, d = 11.5 million, k = 575589, one or two rows in five replaced: 110 us; clearing, applying, averaging and
// stepping in four kernels took 140).
constexpr int kApplyCols = 512;
static_assert(kApplyCols == 1 << kPlusShift, "the message index has this block length");

template <bool STEP>
__global__ __launch_bounds__(kThreads) void plus_apply_long_kernel(PlusLongArgs a, float neg_gamma) {
    constexpr int kPer = kApplyCols / (4 * kWave), kInFlight = 4;
    __shared__ __attribute__((aligned(16))) float lds[kWaves][kApplyCols];
    const int wave = threadIdx.x / kWave, lane = lane_id();
    const int64_t b = (int64_t)blockIdx.x * kWaves + wave;
    if (b >= a.nblk) return;
    float *acc = lds[wave];
    const int64_t c0 = b * kApplyCols, d = a.d, k = a.k;
    const bool whole = c0 + kApplyCols <= d;
    double sum[kPer][4] = {};
    float4 x4[kPer];
    if (STEP && whole) {
#pragma unroll
        for (int q = 0; q < kPer; ++q) x4[q] = *reinterpret_cast<const float4 *>(a.x + c0 + 4 * (q * kWave + lane));
    }
    auto entry = [&](const float *row, int q, int t) {       // of the last, partial block
        const int64_t c = c0 + 4 * (q * kWave + lane) + t;
        return c < d ? row[c] : 0.f;
    };
    for (int32_t w0 = 0; w0 < a.n; w0 += kWave) {
        const int32_t w = w0 + lane;
        const bool plain_l = w < a.n && a.branch[w] != 0;
        const int32_t *start = (plain_l ? a.start_b : a.start_m) + (int64_t)(w < a.n ? w : 0) * (a.nblk + 1) + b;
        const int32_t s0 = w < a.n ? start[0] : 0, s1 = w < a.n ? start[1] : 0;
        const int32_t tile = a.n - w0 < kWave ? a.n - w0 : kWave;
        for (int32_t t0 = 0; t0 < tile; t0 += kInFlight) {
            int32_t e[kInFlight], len[kInFlight];
            int64_t base[kInFlight];
            bool plain[kInFlight];
            float v[kInFlight];
            float4 old[kInFlight][kPer];
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                const int src = t0 + u < tile ? t0 + u : 0;
                const int32_t lo = __shfl(s0, src, kWave), hi = __shfl(s1, src, kWave);
                plain[u] = __shfl((int)plain_l, src, kWave) != 0;
                len[u] = t0 + u < tile ? hi - lo : 0;
                base[u] = (int64_t)(w0 + src) * k + lo;
                const int64_t at = lane < len[u] ? base[u] + lane : 0;     // unconditional loads, no branch
                e[u] = plain[u] ? a.idx_b[at] : a.idx_m[at];
                v[u] = plain[u] ? a.val_b[at] : a.val_m[at];
                const float *row = a.g_i + (int64_t)(w0 + src) * d;
#pragma unroll
                for (int q = 0; q < kPer; ++q) {
                    old[u][q] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (!plain[u]) {
                        if (whole) old[u][q] = load4_any(row + c0 + 4 * (q * kWave + lane));
                        else old[u][q] = make_float4(entry(row, q, 0), entry(row, q, 1), entry(row, q, 2), entry(row, q, 3));
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {            // worker order
                if (t0 + u >= tile) continue;
                float *row = a.g_i + (int64_t)(w0 + t0 + u) * d;
#pragma unroll
                for (int q = 0; q < kPer; ++q) *reinterpret_cast<float4 *>(acc + 4 * (q * kWave + lane)) = old[u][q];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                // line 8 at one position of the run (positions inside a message are distinct)
                auto apply = [&](int32_t pos, float val, int64_t at) {
                    const float now = plain[u] ? val : acc[pos - c0] + val;
                    acc[pos - c0] = now;
                    if (!plain[u]) row[pos] = now;
                    a.msg_idx[at] = pos;
                    a.msg_val[at] = val;
                };
                if (lane < len[u]) apply(e[u], v[u], base[u] + lane);
                for (int32_t j = lane + kWave; j < len[u]; j += kWave) {
                    const int64_t at = base[u] + j;
                    apply(plain[u] ? a.idx_b[at] : a.idx_m[at], plain[u] ? a.val_b[at] : a.val_m[at], at);
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int q = 0; q < kPer; ++q) {
                    const float4 now = *reinterpret_cast<const float4 *>(acc + 4 * (q * kWave + lane));
                    sum[q][0] += (double)now.x;
                    sum[q][1] += (double)now.y;
                    sum[q][2] += (double)now.z;
                    sum[q][3] += (double)now.w;
                    if (plain[u]) {
                        const int64_t c = c0 + 4 * (q * kWave + lane);
                        if (whole) {
                            store4_any(row + c, now);
                        } else {
                            if (c < d) row[c] = now.x;
                            if (c + 1 < d) row[c + 1] = now.y;
                            if (c + 2 < d) row[c + 2] = now.z;
                            if (c + 3 < d) row[c + 3] = now.w;
                        }
                    }
                }
            }
        }
    }
    const double nn = (double)a.n;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int64_t c = c0 + 4 * (q * kWave + lane);
        const float4 g4 = make_float4((float)(sum[q][0] / nn), (float)(sum[q][1] / nn), (float)(sum[q][2] / nn),
                                      (float)(sum[q][3] / nn));
        if (whole) {
            *reinterpret_cast<float4 *>(a.g + c) = g4;
            if (STEP) {
                x4[q].x = fmaf(neg_gamma, g4.x, x4[q].x);
                x4[q].y = fmaf(neg_gamma, g4.y, x4[q].y);
                x4[q].z = fmaf(neg_gamma, g4.z, x4[q].z);
                x4[q].w = fmaf(neg_gamma, g4.w, x4[q].w);
                *reinterpret_cast<float4 *>(a.x + c) = x4[q];
            }
        } else {
            const float gs[4] = {g4.x, g4.y, g4.z, g4.w};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (c + t >= d) continue;
                a.g[c + t] = gs[t];
                if (STEP) a.x[c + t] = fmaf(neg_gamma, gs[t], a.x[c + t]);
            }
        }
    }
}

int64_t chunks_of(int64_t d) { return (d + kNormChunk - 1) / kNormChunk; }
int64_t kept_blocks_of(int64_t k) { return (k + kKeptBlock - 1) / kKeptBlock; }

}  // namespace

size_t plus_scratch_bytes(int32_t n, int64_t d, int64_t k) {
    return sizeof(double2) * (size_t)n * (size_t)(chunks_of(d) + kept_blocks_of(k));
}

size_t plus_long_layout(int32_t n, int64_t d, void *scratch, PlusLong *out) {
    char *base = (char *)scratch;
    const size_t slots = (size_t)n * (size_t)topk_split_slots(n, d), nblk = (size_t)((d + kApplyCols - 1) / kApplyCols);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *p = base ? base + off : nullptr;
        off += (bytes + 255) / 256 * 256;
        return p;
    };
    char *norms = take(sizeof(double2) * slots);
    char *kb = take(sizeof(double) * slots), *km = take(sizeof(double) * slots);
    char *sb = take(sizeof(int32_t) * n * (nblk + 1)), *sm = take(sizeof(int32_t) * n * (nblk + 1));
    if (out) *out = PlusLong{norms, (double *)kb, (double *)km, (int32_t *)sb, (int32_t *)sm, (int64_t)nblk};
    return off;
}

namespace {
// Line 8 in two kernels: rows whose worker chose the plain compressor are cleared, the chosen pairs applied.
void launch_apply_rows(const int32_t *branch, float *g_i, int32_t n, int64_t d, int64_t k, const int32_t *idx_b,
                       const float *val_b, const int32_t *idx_m, const float *val_m, int32_t *msg_idx, float *msg_val,
                       hipStream_t stream) {
    const dim3 grid((unsigned)chunks_of(d), (unsigned)n);
    if (d % 4 == 0 && (uintptr_t)g_i % 16 == 0)      // kNormChunk is a multiple of four: every chunk is whole float4s
        hipLaunchKernelGGL(plus_clear_kernel<4>, grid, dim3(kThreads), 0, stream, branch, g_i, d);
    else
        hipLaunchKernelGGL(plus_clear_kernel<1>, grid, dim3(kThreads), 0, stream, branch, g_i, d);
    int64_t blocks = (k + kThreads - 1) / kThreads;
    if (blocks > 256) blocks = 256;
    hipLaunchKernelGGL(plus_apply_kernel, dim3((unsigned)blocks, (unsigned)n), dim3(kThreads), 0, stream, branch,
                       idx_b, val_b, idx_m, val_m, k, msg_idx, msg_val, g_i, d);
}
}  // namespace

// Many workers and few blocks of coordinates: plus_apply_long_kernel takes a wavefront per block and worker after worker,
// so line 8 goes over the rows instead, and lines 10 and 3 are kernels of their own.  step, us, by coordinates and by rows:
// 20 x 60000 41 and 43; 32 x 60000 48 and 46; 32 x 250000 66 and 69; 64 x 100000 81 and 67; 100 x 250000 126 and 130;
// 200 x 60000 149 and 92; 1000 x 17000 598 and 285.
hipError_t launch_plus_long(const PlusLong &pl, PlusLongArgs a, double *BM, float gamma, hipStream_t stream) {
    if (((uintptr_t)a.g | (uintptr_t)(a.x ? a.x : a.g)) % 16 != 0) return hipErrorInvalidValue;
    a.start_b = pl.start_plain;
    a.start_m = pl.start_markov;
    a.nblk = pl.nblk;
    hipLaunchKernelGGL(plus_decide_long_kernel, dim3((unsigned)a.n), dim3(kThreads), 0, stream, (const double2 *)pl.norms,
                       pl.kept_plain, pl.kept_markov, topk_split_slots(a.n, a.d), a.branch, BM);
    if (a.n >= 32 && a.d <= 200000) {
        launch_apply_rows(a.branch, a.g_i, a.n, a.d, a.k, a.idx_b, a.val_b, a.idx_m, a.val_m, a.msg_idx, a.msg_val, stream);
        hipError_t st = launch_mean_rows(a.g_i, a.g, a.n, a.d, stream);
        if (st == hipSuccess && a.x) st = launch_model_step(a.x, a.g, a.d, gamma, stream);
        return st;
    }
    const dim3 grid((unsigned)((a.nblk + kWaves - 1) / kWaves)), block(kThreads);
    if (a.x) hipLaunchKernelGGL(plus_apply_long_kernel<true>, grid, block, 0, stream, a, -gamma);
    else hipLaunchKernelGGL(plus_apply_long_kernel<false>, grid, block, 0, stream, a, -gamma);
    return hipGetLastError();
}

hipError_t launch_plus_choose(const float *s, float *g_i, int32_t n, int64_t d, int64_t k, const int32_t *idx_b,
                              const float *val_b, const int32_t *idx_m, const float *val_m, void *scratch,
                              int32_t *branch, double *BM, int32_t *msg_idx, float *msg_val, hipStream_t stream) {
    const int64_t chunks = chunks_of(d);
    double2 *part = (double2 *)scratch;
    // kNormChunk is a multiple of four, so with d % 4 == 0 every chunk is whole float4s
    const bool vec4 = (d % 4 == 0) && (((uintptr_t)s | (uintptr_t)g_i) % 16 == 0);
    if (vec4) {
        hipLaunchKernelGGL(plus_sqnorms_kernel<4>, dim3((unsigned)chunks, (unsigned)n), dim3(kThreads), 0, stream, s,
                           g_i, d, part);
    } else {
        hipLaunchKernelGGL(plus_sqnorms_kernel<1>, dim3((unsigned)chunks, (unsigned)n), dim3(kThreads), 0, stream, s,
                           g_i, d, part);
    }
    const int64_t kblocks = k <= kKeptBlock ? 0 : kept_blocks_of(k);     // short messages: summed by the decide kernel
    double2 *kept = part + (size_t)n * chunks;
    if (kblocks > 0)
        hipLaunchKernelGGL(plus_kept_kernel, dim3((unsigned)kblocks, (unsigned)n), dim3(kThreads), 0, stream, s, g_i,
                           d, val_b, idx_m, k, kept);
    hipLaunchKernelGGL(plus_decide_kernel, dim3((unsigned)n), dim3(kThreads), 0, stream, part, chunks, kept, kblocks, s,
                       g_i, d, val_b, idx_m, k, branch, BM);
    launch_apply_rows(branch, g_i, n, d, k, idx_b, val_b, idx_m, val_m, msg_idx, msg_val, stream);
    return hipGetLastError();
}

}  // namespace ef21
