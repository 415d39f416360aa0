// The power iteration of ef21_theory_stepsize on the workers' Gram matrices G_i = (1/m) A_i^T A_i (d x d), for dense
// problems with few columns.  Iterating with A reads the whole problem twice per iteration (once for the workers'
// vectors, once for the common one) in six launches; G_i is formed once per call on the matrix cores and an iteration
// is then a d x d product.
//
//   gram_tile     G_i in tiles of 32 x 32 on and above the diagonal: v_mfma_f64_16x16x4, products of the fp32 entries
//                 and their sums in fp64.  Rows are cut into chunks so that the chip is full; four wavefronts of a
//                 workgroup share a chunk.
//   gram_finish   the chunks added, divided by m, rounded to fp32 once and written to both halves; one more matrix is
//                 the mean over the workers, G = (1/(nm)) sum_i A_i^T A_i.
//   The estimate after T iterations is sqrt(u_2T / u_2T-2), u_N = v' G^N v with the start vector v.  Between 48 and 2822
//   iterations these moments come from J = ceil(4.8 sqrt(T)) + 1 steps of the Lanczos recurrence instead (49 products
//   with G in the place of 100 at T = 100): u_N / |v|^2 is entry (1, 1) of the N-th power of its J x J tridiagonal matrix, exactly for
//   N < 2J and to twice the error of the best polynomial of degree 2J - 1 on [0, lambda_max] beyond; for t^N that is at most
//   2 exp(-4 J^2 / N) (Newman and Rivlin, Approximation of monomials by lower degree polynomials, 1976): 2e-20 of
//   lambda_max^N.  What loss of orthogonality adds is rounding (Druskin and Knizhnerman, Error bounds in the simple Lanczos
//   procedure, 1991): the tests hold the estimates against the power iteration in fp64 from the same
//   start vector on Gaussian, non-negative, rank-three, rank-one, badly scaled and diagonal matrices, where what is
//   left is the start vector's rounding to fp32 (2^-23).
//   The T iterations are then taken with the tridiagonal matrix, by one wavefront.  n = 20, m = 2487, d = 300, 100
//   iterations: 436 -> 319 us a call;
//   n = 2, m = 7500, d = 1000: 1255 -> 800.
//   Where that is the faster way the start vector is taken to y = G^(T-1) v by squarings instead, G^2, G^4, .., G^(2^s) in fp64 (gram_square;
//   two products a step have to wait for each other, the 21 x 300^3 of a square have the whole chip), and applications of those powers,
//   and the estimate is |G y| / |y|.  A relative error e of a power becomes 2 e in its square, some 2^s of a rounding in all, in y alone: the
//   last product is taken with G itself.  n = 20, m = 2487, d = 300: 317 -> 289 us a call of 100 iterations, 660 -> 363 of 1000; 32, 1400, 330
//   563 -> 373; 3, 2000, 700 528 -> 325; 2, 7500, 1000 796 -> 656.
//   d <= 320:     ONE launch runs all iterations, a workgroup of 1024 threads per matrix.  G sits in registers (a
//                 compute unit has 512 KB of them: 100 entries per thread at d = 320), the vector in LDS; a wavefront
//                 multiplies its rows of G (columns, by symmetry) and the sixteen partial vectors are added in LDS.
//   d <= 1024:    a launch per iteration; every workgroup works out the vector of the recurrence for itself (d entries)
//                 and multiplies 32 rows of G.
// Vectors, products with G, sums and norms are in fp64; G is the only thing rounded to fp32, so the constants are
// closer to the exact ones than through fp32 products with A.
#include <algorithm>
#include <cmath>
#include <utility>

#include "device_utils.h"
#include "gram_way.h"
#include "kernels.h"

namespace ef21 {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kTileThreads = 256, kTileWaves = kTileThreads / kWave;
constexpr int kStepRows = 4;                         // rows of A per matrix instruction
constexpr int kAhead = 4;                            // instructions' rows whose loads are in flight

constexpr int kResThreads = 1024, kResWaves = kResThreads / kWave;
constexpr int32_t kItersPerLaunch = 4096;            // of the resident kernel: bounds a launch to some ten milliseconds

constexpr int kMvThreads = 256, kMvWaves = kMvThreads / kWave, kMvRowsPerWave = 8;
constexpr int kMvRows = kMvWaves * kMvRowsPerWave;
static_assert(kMvRows == kTile, "G is padded to whole tiles, so a workgroup's rows all exist");

// tile number -> (I, J), I <= J: J (J + 1) / 2 + I
__device__ __forceinline__ void tile_of(int32_t pair, int32_t *I, int32_t *J) {
    int32_t j = (int32_t)((sqrtf(8.0f * (float)pair + 1.0f) - 1.0f) * 0.5f);
    while (j * (j + 1) / 2 > pair) --j;
    while ((j + 1) * (j + 2) / 2 <= pair) ++j;
    *J = j;
    *I = pair - j * (j + 1) / 2;
}

// part[worker][chunk][pair][32][32] = sum over the chunk's rows of a_l[I's columns] a_l[J's columns]^T.
// Operand of v_mfma_f64_16x16x4: lane j holds row j / 16 of the four and column j % 16 of the sixteen; result
// register v of lane j is entry (j / 16 + 4 v, j % 16).  Bound by the matrix cores: four instructions (256 clocks of a
// SIMD) per four loads of 64-byte pieces, whose addresses are a scalar base and a constant offset per lane.  Columns
// past d repeat column 0; what they add up to is dropped by gram_finish_kernel.
__global__ __launch_bounds__(kTileThreads) void gram_tile_kernel(const float *__restrict__ A, int64_t m, int64_t d,
                                                                 int64_t rows_per_chunk, int64_t chunks, int64_t units,
                                                                 int64_t pairs, double *__restrict__ part) {
    __shared__ double red[kTileWaves][kTileEntries];
    // all tiles of a unit (a worker's chunk of rows) on one XCD: its L2 then fetches the rows once
    const int64_t turn = blockIdx.x / kXcds, unit = turn / pairs * kXcds + blockIdx.x % kXcds;
    if (unit >= units) return;                       // the whole workgroup
    const int64_t pair = turn % pairs, chunk = unit % chunks, worker = unit / chunks;
    const int wave = threadIdx.x / kWave, lane = lane_id();
    int32_t I, J;
    tile_of((int32_t)pair, &I, &J);
    const int64_t l0 = chunk * rows_per_chunk;
    const int64_t rows = l0 + rows_per_chunk < m ? rows_per_chunk : m - l0;
    // matrix instruction s of a wavefront takes rows 16 s + 4 wave .. of the chunk
    constexpr int kStride = kTileWaves * kStepRows;
    const char *base = reinterpret_cast<const char *>(A + (worker * m + l0) * d);
    const int32_t my_row = wave * kStepRows + lane / 16;
    uint32_t off[4];                                 // bytes: two groups of sixteen columns of I, two of J
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int32_t c = (t < 2 ? I : J) * kTile + (t & 1) * 16 + (lane & 15);
        off[t] = 4u * (uint32_t)(my_row * (int32_t)d + (c < d ? c : 0));
    }
    const int64_t step_bytes = 4 * kStride * d;
    v4d acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = (v4d){0.0, 0.0, 0.0, 0.0};
    auto multiply = [&](const float (&v)[4]) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)v[i], (double)v[2 + j], acc[i][j], 0, 0, 0);
    };
    const int64_t groups = rows / (kAhead * kStride);           // of kAhead instructions, all rows inside the chunk
    auto load_group = [&](int64_t g, float (&v)[kAhead][4]) {
        const char *p = base + g * kAhead * step_bytes;
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
#pragma unroll
            for (int t = 0; t < 4; ++t) v[u][t] = *reinterpret_cast<const float *>(p + u * step_bytes + off[t]);
    };
    if (groups > 0) {
        float v[kAhead][4], next[kAhead][4];
        load_group(0, v);
        for (int64_t g = 0; g < groups; ++g) {
            load_group(g + 1 < groups ? g + 1 : g, next);
#pragma unroll
            for (int u = 0; u < kAhead; ++u) multiply(v[u]);
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
#pragma unroll
                for (int t = 0; t < 4; ++t) v[u][t] = next[u][t];
        }
    }
    for (int64_t r0 = groups * kAhead * kStride; r0 < rows; r0 += kStride) {      // the rest; a row past the chunk is zero
        const bool live = r0 + my_row < rows;
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            v[t] = *reinterpret_cast<const float *>(base + (live ? r0 * d * 4 + off[t] : 0));
            if (!live) v[t] = 0.f;
        }
        multiply(v);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                red[wave][(i * 16 + lane / 16 + 4 * r) * kTile + j * 16 + (lane & 15)] = acc[i][j][r];
    __syncthreads();
    double *out = part + (unit * pairs + pair) * kTileEntries;
    for (int e = threadIdx.x; e < kTileEntries; e += kTileThreads)
        out[e] = ((red[0][e] + red[1][e]) + red[2][e]) + red[3][e];
}

// Matrix `which` of n + 1 (the last one: the mean over the workers): the partial sums in order, scaled, rounded to fp32 once.
// Where the entries are kept in fp64 the tiles on the diagonal leave their sum of diagonal entries in traces[matrix][tile].
template <class T>
__global__ __launch_bounds__(kTileThreads) void gram_finish_kernel(const double *__restrict__ part, int64_t chunks,
                                                                   int64_t pairs, int64_t d, int64_t ld, double m,
                                                                   T *__restrict__ G, double *__restrict__ traces) {
    constexpr int kPer = kTileEntries / kTileThreads, kInFlight = 4;
    __shared__ T tile[kTile][kTile + 1];
    const int64_t pair = blockIdx.x, which = blockIdx.y, n = gridDim.y - 1;
    const bool mean = which == n;
    const int64_t count = mean ? n * chunks : chunks;
    const double *src = part + ((mean ? 0 : which * chunks) * pairs + pair) * kTileEntries;
    double s[kPer] = {};
    for (int64_t b = 0; b < count; b += kInFlight) {
        double v[kInFlight][kPer];
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            const int64_t at = b + u < count ? b + u : b;
#pragma unroll
            for (int q = 0; q < kPer; ++q) v[u][q] = src[at * pairs * kTileEntries + threadIdx.x + q * kTileThreads];
        }
#pragma unroll
        for (int u = 0; u < kInFlight; ++u)
#pragma unroll
            for (int q = 0; q < kPer; ++q) s[q] += b + u < count ? v[u][q] : 0.0;
    }
    const double scale = mean ? m * (double)n : m;
    int32_t I, J;
    tile_of((int32_t)pair, &I, &J);
    T *out = G + which * ld * ld;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int e = threadIdx.x + q * kTileThreads, r = e / kTile, c = e % kTile;
        const float g = I * kTile + r < d && J * kTile + c < d ? (float)(s[q] / scale) : 0.f;
        tile[r][c] = (T)g;
        out[((int64_t)I * kTile + r) * ld + (int64_t)J * kTile + c] = (T)g;
    }
    if (I == J && sizeof(T) == 4) return;            // symmetric by itself (the products commute)
    __syncthreads();
    if (I == J) {
        if (threadIdx.x == 0) {
            double sum = 0.0;
            for (int i = 0; i < kTile; ++i) sum += (double)tile[i][i];
            traces[which * kTraces + I] = sum;
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int e = threadIdx.x + q * kTileThreads, r = e / kTile, c = e % kTile;
        out[((int64_t)J * kTile + r) * ld + (int64_t)I * kTile + c] = tile[c][r];
    }
}

// Sum over each group of LANES consecutive lanes (16 or 64), as group_sum does it: no trip through the LDS crossbar.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
template <int LANES>
__device__ __forceinline__ double group_sum_f64(double v) {
    static_assert(LANES == 16 || LANES == 64, "whole rows of sixteen lanes");
    v += dpp_f64<0xB1>(v);                  // quad_perm [1,0,3,2]
    v += dpp_f64<0x4E>(v);                  // quad_perm [2,3,0,1]
    v += dpp_f64<0x141>(v);                 // row_half_mirror
    v += dpp_f64<0x140>(v);                 // row_mirror
    if constexpr (LANES == 64) {
        const uint32_t lo = (uint32_t)__double2loint(v), hi = (uint32_t)__double2hiint(v);
        const auto l16 = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto h16 = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        v = __hiloint2double((int)h16[0], (int)l16[0]) + __hiloint2double((int)h16[1], (int)l16[1]);
        const uint32_t lo2 = (uint32_t)__double2loint(v), hi2 = (uint32_t)__double2hiint(v);
        const auto l32 = __builtin_amdgcn_permlane32_swap(lo2, lo2, false, false);
        const auto h32 = __builtin_amdgcn_permlane32_swap(hi2, hi2, false, false);
        v = __hiloint2double((int)h32[0], (int)l32[0]) + __hiloint2double((int)h32[1], (int)l32[1]);
    }
    return v;
}
__device__ __forceinline__ double wave_sum_f64(double v) { return group_sum_f64<kWave>(v); }

// v[row][0..ld): the start vectors (zero past d)
__global__ __launch_bounds__(kTileThreads) void gram_start_kernel(double *__restrict__ v, int64_t d, int64_t ld) {
    const int64_t row = blockIdx.y, j = (int64_t)blockIdx.x * kTileThreads + threadIdx.x;
    if (j < ld) v[row * ld + j] = j < d ? (double)power_start_entry(row, j, rsqrtf((float)d)) : 0.0;
}

// 1 / |w|, or 0 for w = 0 (the vector then stays zero, as do the norms that follow)
__device__ __forceinline__ double inverse_norm(double sum_sq) { return sum_sq == 0.0 ? 0.0 : 1.0 / sqrt(sum_sq); }

// x of the next lower / next higher lane, zero at the end of the wavefront
__device__ __forceinline__ double from_lower(double x) { return dpp_f64<0x138>(x); }    // wave_shr:1
__device__ __forceinline__ double from_higher(double x) { return dpp_f64<0x130>(x); }   // wave_shl:1

// What `iterations` steps of the power iteration from the first unit vector give for the symmetric tridiagonal matrix with
// diagonal alpha[0..steps) and beta[i] beside it in rows i - 1 and i; by one wavefront, PER rows per lane.  The vector is
// scaled every 32 steps (the matrix has a trace of about one, so its largest eigenvalue is at least 1 / (2 d)).
template <int PER>
__device__ double tridiagonal_power(const double *alpha, const double *beta, int32_t steps, int32_t iterations) {
    const int lane = lane_id();
    double a[PER], b[PER + 1], y[PER];
#pragma unroll
    for (int q = 0; q <= PER; ++q) {
        const int i = lane * PER + q;
        if (q < PER) {
            a[q < PER ? q : 0] = i < steps ? alpha[i] : 0.0;
            y[q < PER ? q : 0] = i == 0 ? 1.0 : 0.0;
        }
        b[q] = i > 0 && i < steps ? beta[i] : 0.0;
    }
    auto length_sq = [&]() {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < PER; ++q) s += y[q] * y[q];
        return wave_sum_f64(s);
    };
    auto multiply = [&]() {
        const double below = from_lower(y[PER - 1]), above = from_higher(y[0]);
        double z[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q)
            z[q] = fma(b[q], q > 0 ? y[q > 0 ? q - 1 : 0] : below, fma(b[q + 1], q + 1 < PER ? y[q + 1 < PER ? q + 1 : 0] : above, a[q] * y[q]));
#pragma unroll
        for (int q = 0; q < PER; ++q) y[q] = z[q];
    };
    for (int32_t it = 1; it < iterations; ++it) {
        multiply();
        if (it % 32 == 0 || it + 1 == iterations) {
            const double inv = inverse_norm(length_sq());
#pragma unroll
            for (int q = 0; q < PER; ++q) y[q] *= inv;
        }
    }
    multiply();                                      // of a unit vector, or zero
    return sqrt(length_sq());
}

// All iterations of one matrix.  NC: columns / 64.  w (one entry per thread) is the product of the iteration before,
// w = G w' / |w'|, whose length is the estimate; the division happens after the product, so that an iteration holds two
// barriers.  G is scaled by a power of two to a trace of about one (products of G with w are of the order of its
// square).  fp32 products were measured too (1.8 us an iteration at d = 300 against 2.9): where the top eigenvalues nearly
// coincide the constants then end up further from the exact ones than by iterating with A.
// state [matrix][ld]: w between launches.
// LANCZOS: `steps` steps of the recurrence w = G v_j - alpha_j v_j - beta_j v_{j-1}, v_{j+1} = w / |w| instead (one launch,
// first), the division put off in the same way; alpha_j = v_j' G v_j is summed from the wavefronts' products beside them.
template <int NC, bool LANCZOS>
__global__ __launch_bounds__(kResThreads) void gram_resident_kernel(const float *__restrict__ G, int64_t d, int64_t ld,
                                                                    int32_t iterations, int32_t steps, bool first,
                                                                    double *__restrict__ state,
                                                                    double2 *__restrict__ stats) {
    constexpr int kCols = NC * kWave, NR = kCols / kResWaves;        // rows of G per wavefront
    constexpr int kLds = NC >= 4 ? 4 : 0, kReg = NR - kLds;          // four of the rows in LDS, or registers spill
    static_assert(kReg % 2 == 0 && (kLds == 0 || kLds == 4), "rows go in pairs, those in LDS as one float4 per column");
    __shared__ double part[kResWaves][kCols], sums[kResWaves];
    __shared__ __attribute__((aligned(16))) double vec[kCols];
    __shared__ float4 g_lds[kLds ? kResWaves : 1][kLds ? kCols : 1];
    __shared__ double prev[LANCZOS ? kCols : 1], dots[LANCZOS ? kResWaves : 1];
    __shared__ double alpha[LANCZOS ? kLanczosMax : 1], beta[LANCZOS ? kLanczosMax : 1];
    const int tid = threadIdx.x, wave = wave_id(), lane = lane_id();
    const float *g = G + (int64_t)blockIdx.x * ld * ld;
    // sum over the workgroup of the threads below kCols (whole wavefronts; the others pass zeros)
    auto norm_part = [&](double x) {
        if (tid < kCols) {
            const double s = wave_sum_f64(x);
            if (lane == 0) sums[wave] = s;
        }
    };
    auto total = [&]() {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < NC; ++q) s += sums[q];
        return s;
    };
    norm_part(tid < ld ? (double)g[(int64_t)tid * ld + tid] : 0.0);
    __syncthreads();
    const double trace = total();
    int exponent = 0;
    if (trace > 0.0 && trace < 1e300) (void)frexp(trace, &exponent);
    const float scale = ldexpf(1.0f, -exponent > 126 ? 126 : (-exponent < -126 ? -126 : -exponent));
    float gr[kReg][NC];
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const int r = wave * NR + i, c = lane + j * kWave;
            const float e = r < ld && c < ld ? g[(int64_t)r * ld + c] * scale : 0.f;
            if (i < kReg) gr[i < kReg ? i : 0][j] = e;
            else reinterpret_cast<float *>(&g_lds[kLds ? wave : 0][kLds ? c : 0])[i - kReg] = e;   // read by the same lane only
        }
    double *vr = state + (int64_t)blockIdx.x * ld;
    double w = 0.0;
    if (first) w = tid < d ? (double)power_start_entry(blockIdx.x, tid, rsqrtf((float)d)) : 0.0;
    else if (tid < ld) w = vr[tid];
    if (LANCZOS && tid < kCols) prev[LANCZOS ? tid : 0] = 0.0;
    __syncthreads();                                 // the trace has been read
    const int32_t rounds = LANCZOS ? steps : iterations;
    for (int32_t it = 0; it < rounds; ++it) {
        norm_part(w * w);
        if (tid < kCols) vec[tid] = w;
        __syncthreads();
        double acc[NC] = {};
#pragma unroll
        for (int i = 0; i < kReg; i += 2) {          // LDS reads cost as much as the products: two entries at a time
            const double2 x = *reinterpret_cast<const double2 *>(vec + wave * NR + i);
#pragma unroll
            for (int j = 0; j < NC; ++j) {           // converted here: hoisted out of the loop, G would take twice the
                asm("" : "+v"(gr[i][j]), "+v"(gr[i + 1][j]));                    // registers
                acc[j] = fma((double)gr[i][j], x.x, acc[j]);
                acc[j] = fma((double)gr[i + 1][j], x.y, acc[j]);
            }
            __builtin_amdgcn_sched_barrier(0);       // no more than two rows' operands at a time
        }
        if constexpr (kLds != 0) {
            const double2 x0 = *reinterpret_cast<const double2 *>(vec + wave * NR + kReg);
            const double2 x1 = *reinterpret_cast<const double2 *>(vec + wave * NR + kReg + 2);
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                const float4 e = g_lds[wave][lane + j * kWave];
                acc[j] = fma((double)e.x, x0.x, acc[j]);
                acc[j] = fma((double)e.y, x0.y, acc[j]);
                acc[j] = fma((double)e.z, x1.x, acc[j]);
                acc[j] = fma((double)e.w, x1.y, acc[j]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) part[wave][lane + j * kWave] = acc[j];
        if constexpr (LANCZOS) {                     // this wavefront's rows' share of w' G w
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                __builtin_amdgcn_sched_barrier(0);
                s = fma(acc[j], vec[lane + j * kWave], s);
            }
            s = wave_sum_f64(s);
            if (lane == 0) dots[wave] = s;
        }
        double inv = 0.0, length_sq = 0.0;
        if (tid < kCols) {
            length_sq = total();
            inv = inverse_norm(length_sq);
        }
        __syncthreads();
        if (tid < kCols) {
            double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll
            for (int q = 0; q < kResWaves; q += 4) {
                if (LANCZOS && q == kResWaves / 2) __builtin_amdgcn_sched_barrier(0);
                s0 += part[q][tid];
                s1 += part[q + 1][tid];
                s2 += part[q + 2][tid];
                s3 += part[q + 3][tid];
            }
            w = ((s0 + s1) + (s2 + s3)) * inv;
            if constexpr (LANCZOS) {                 // w = G v_j so far, v_j = vec * inv
                __builtin_amdgcn_sched_barrier(0);   // the sixteen shares after the sixteen partial products, not beside them
                static_assert(kResWaves == 16, "one row of lanes");
                const double al = group_sum_f64<kResWaves>(dots[lane % kResWaves]) * inv * inv, be = sqrt(length_sq), v = vec[tid] * inv;
                w = fma(-be, prev[tid], fma(-al, v, w));     // prev = 0 the first time, when be is the start vector's length
                prev[tid] = v;
                alpha[it] = al;                      // the same from every thread: behind a branch the loop's registers spill
                beta[it] = be;
            }
        }
    }
    if constexpr (LANCZOS) {
        __syncthreads();
        if (wave > 0) return;
        const double value = steps <= kWave ? tridiagonal_power<1>(alpha, beta, steps, iterations)
                                            : tridiagonal_power<kLanczosMax / kWave>(alpha, beta, steps, iterations);
        if (lane == 0) stats[blockIdx.x] = make_double2(0.0, value / (double)scale);
        return;
    }
    if (tid < ld) vr[tid] = w;
    norm_part(w * w);                                // stats[matrix] = (0, the estimate)
    __syncthreads();
    if (tid == 0) stats[blockIdx.x] = make_double2(0.0, sqrt(total()) / (double)scale);
}

// One iteration: w = G v / |v|.  Grid (ld / 32, matrices).
// Recurrence number `step` of the Lanczos path (step >= 0): v is the product G v_j (step 0: the start vector), r.vj and
// r.vprev are v_j and the one before; every workgroup forms v_{j+1} for itself and multiplies its rows, and the first one of
// a matrix leaves alpha_j, beta_{j+1} and v_{j+1} for the launches that follow.
struct Recurrence {
    int32_t step;                                    // -1: the power iteration
    const double *vj, *vprev;                        // [matrix][ld]
    double *vnext;
    double *alpha, *beta;                            // [matrix][kLanczosMax]
};
__global__ __launch_bounds__(kMvThreads) void gram_matvec_kernel(const float *__restrict__ G, int64_t ld,
                                                                 const double *__restrict__ v, double *__restrict__ w,
                                                                 Recurrence r) {
    constexpr int kMaxPer = (int)kGramMax / kMvThreads, kQuads = (int)kGramMax / (4 * kWave), kTogether = 2;
    __shared__ double vec[kGramMax], sums[2][kMvWaves];
    const int64_t which = blockIdx.y;
    const int tid = threadIdx.x, wave = tid / kWave, lane = lane_id();
    const double *vr = v + which * ld;
    auto block_sum = [&](double s, int slot) {
        s = wave_sum_f64(s);
        if (lane == 0) sums[slot][wave] = s;
        __syncthreads();
        s = 0.0;
#pragma unroll
        for (int q = 0; q < kMvWaves; ++q) s += sums[slot][q];
        return s;
    };
    double x[kMaxPer], sq = 0.0;
#pragma unroll
    for (int q = 0; q < kMaxPer; ++q) {
        const int j = tid + q * kMvThreads;
        x[q] = j < ld ? vr[j] : 0.0;
    }
    if (r.step > 0) {
        double vj[kMaxPer], vp[kMaxPer], dot = 0.0;
        const double be = r.beta[which * kLanczosMax + r.step - 1];
#pragma unroll
        for (int q = 0; q < kMaxPer; ++q) {
            const int j = tid + q * kMvThreads;
            vj[q] = j < ld ? r.vj[which * ld + j] : 0.0;
            vp[q] = r.step > 1 && j < ld ? r.vprev[which * ld + j] : 0.0;
            dot = fma(x[q], vj[q], dot);
        }
        dot = block_sum(dot, 0);
#pragma unroll
        for (int q = 0; q < kMaxPer; ++q) x[q] = fma(-be, vp[q], fma(-dot, vj[q], x[q]));
        if (blockIdx.x == 0 && tid == 0) r.alpha[which * kLanczosMax + r.step - 1] = dot;
    }
#pragma unroll
    for (int q = 0; q < kMaxPer; ++q) sq += x[q] * x[q];
    sq = block_sum(sq, 1);
    const double inv = inverse_norm(sq);
#pragma unroll
    for (int q = 0; q < kMaxPer; ++q) {
        const int j = tid + q * kMvThreads;
        vec[j] = x[q] * inv;
        if (r.step >= 0 && blockIdx.x == 0 && j < ld) r.vnext[which * ld + j] = x[q] * inv;
    }
    if (r.step >= 0 && blockIdx.x == 0 && tid == 0) r.beta[which * kLanczosMax + r.step] = r.step > 0 ? sqrt(sq) : 0.0;
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * kMvRows + wave * kMvRowsPerWave;
    const float *g = G + (which * ld + r0) * ld;
#pragma unroll
    for (int i0 = 0; i0 < kMvRowsPerWave; i0 += kTogether) {
        float4 a[kTogether][kQuads];
#pragma unroll
        for (int i = 0; i < kTogether; ++i)
#pragma unroll
            for (int q = 0; q < kQuads; ++q) {
                const int64_t c = 4 * (lane + q * kWave);            // ld is a multiple of 32
                a[i][q] = c < ld ? *reinterpret_cast<const float4 *>(g + (i0 + i) * ld + c) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
        for (int i = 0; i < kTogether; ++i) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < kQuads; ++q) {
                const int c = 4 * (lane + q * kWave);
                s = fma((double)a[i][q].x, vec[c], s);
                s = fma((double)a[i][q].y, vec[c + 1], s);
                s = fma((double)a[i][q].z, vec[c + 2], s);
                s = fma((double)a[i][q].w, vec[c + 3], s);
            }
            s = wave_sum_f64(s);
            if (lane == 0) w[which * ld + r0 + i0 + i] = s;
        }
    }
}

// stats[row] = (0, |w|): what the last iteration multiplied was a unit vector.  One wavefront per row.
__global__ __launch_bounds__(kWave) void gram_norm_kernel(const double *__restrict__ w, int64_t ld,
                                                          double2 *__restrict__ stats) {
    const double *r = w + (int64_t)blockIdx.x * ld;
    double s = 0.0;
    for (int64_t j = threadIdx.x; j < ld; j += kWave) s += r[j] * r[j];
    s = wave_sum_f64(s);
    if (threadIdx.x == 0) stats[blockIdx.x] = make_double2(0.0, sqrt(s));
}

// The end of the Lanczos path: the last alpha, then the power iteration with the tridiagonal matrix.  y = G v_J.
__global__ __launch_bounds__(kWave) void gram_tridiagonal_kernel(const double *__restrict__ y, const double *__restrict__ v,
                                                                 int64_t ld, const double *__restrict__ alpha,
                                                                 const double *__restrict__ beta, int32_t steps,
                                                                 int32_t iterations, double2 *__restrict__ stats) {
    __shared__ double a[kLanczosMax], b[kLanczosMax];
    const int64_t which = blockIdx.x;
    const int lane = lane_id();
    double dot = 0.0, trace = 0.0;
    for (int64_t j = lane; j < ld; j += kWave) dot = fma(y[which * ld + j], v[which * ld + j], dot);
    dot = wave_sum_f64(dot);
    for (int32_t i = lane; i < steps; i += kWave) {
        a[i] = i + 1 < steps ? alpha[which * kLanczosMax + i] : dot;
        b[i] = beta[which * kLanczosMax + i];
        trace += a[i];
    }
    trace = wave_sum_f64(trace);
    int exponent = 0;                                // scaled as in gram_resident_kernel; every eigenvalue is in [0, trace]
    if (trace > 0.0 && trace < 1e300) (void)frexp(trace, &exponent);
    for (int32_t i = lane; i < steps; i += kWave) {
        a[i] = ldexp(a[i], -exponent);
        b[i] = ldexp(b[i], -exponent);
    }
    __syncthreads();
    const double value = steps <= kWave ? tridiagonal_power<1>(a, b, steps, iterations)
                                        : tridiagonal_power<kLanczosMax / kWave>(a, b, steps, iterations);
    if (lane == 0) stats[which] = make_double2(0.0, ldexp(value, exponent));
}

// ---- powers of G by squaring
// M, in fp64 and symmetric, [n + 1][ld][ld], stands for its multiple with a trace in [1/2, 1): every kernel that reads it
// multiplies by that power of two, which is exact.  Its trace is the sum of the first `parts` entries of traces[matrix].
// Of that multiple the largest eigenvalue lies between 1 / (2 d) (all d alike: columns that are orthogonal and of one length) and 1, and
// nothing rescales the vector, so its products are taken with `lift` times the multiple, the power of two next above sqrt(d): they grow or
// shrink by at most 2^6 each.  There are sixty of them at most (a call that needs c applications beyond the squarings has c at most twice
// the ratio of the two times, 40, and twenty bits), so that the squares of the entries stay within 2^(+-800).
struct Power {
    const double *M, *traces;
    int32_t parts;
    double lift;
};
// 2^-e, the trace being in [2^(e-1), 2^e); the same in all lanes
__device__ __forceinline__ double unit_scale(double part_of_trace) {
    const double trace = wave_sum_f64(part_of_trace);
    int exponent = 0;
    if (trace > 0.0 && trace < 1e300) (void)frexp(trace, &exponent);
    return ldexp(1.0, -exponent);
}
__device__ __forceinline__ double trace_part(const Power &a, int64_t which) {
    return lane_id() < a.parts ? a.traces[which * kTraces + lane_id()] : 0.0;
}

// z = M y for rows [r0, r0 + 32) of matrix `which`, of whose columns `cols` are used (the squares leave those beyond unwritten);
// y == nullptr: the start vector.  vec: LDS.  A wavefront's eight rows, TOGETHER of them in flight, PAIRS x 128 columns at most.
template <int PAIRS, int TOGETHER>
__device__ __forceinline__ void power_rows(const Power &a, int64_t which, int64_t r0, int64_t d, int64_t cols, int64_t ld,
                                           const double *__restrict__ y, double *__restrict__ z, double *vec) {
    const int tid = threadIdx.x, wave = tid / kWave, lane = lane_id();
    const double part = trace_part(a, which);
    const double *g = a.M + (which * ld + r0 + wave * kMvRowsPerWave) * ld;
    double2 m[TOGETHER][PAIRS];
    auto load = [&](int i0) {
#pragma unroll
        for (int i = 0; i < TOGETHER; ++i)
#pragma unroll
            for (int q = 0; q < PAIRS; ++q) {
                const int64_t c = 2 * (lane + q * kWave);
                m[i][q] = c < cols ? *reinterpret_cast<const double2 *>(g + (i0 + i) * ld + c) : make_double2(0.0, 0.0);
            }
    };
    load(0);
    for (int64_t j = tid; j < PAIRS * 2 * kWave; j += kMvThreads)
        vec[j] = j >= cols ? 0.0 : y ? y[which * ld + j] : j < d ? (double)power_start_entry(which, j, rsqrtf((float)d)) : 0.0;
    __syncthreads();
    const double scale = a.lift * unit_scale(part);
#pragma unroll
    for (int i0 = 0; i0 < kMvRowsPerWave; i0 += TOGETHER) {
        if (i0 > 0) load(i0);
#pragma unroll
        for (int i = 0; i < TOGETHER; ++i) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < PAIRS; ++q) {
                const int c = 2 * (lane + q * kWave);
                s = fma(m[i][q].x, vec[c], fma(m[i][q].y, vec[c + 1], s));
            }
            s = wave_sum_f64(s);
            const int64_t row = r0 + wave * kMvRowsPerWave + i0 + i;
            if (lane == 0) z[which * ld + row] = row < cols ? s * scale : 0.0;
        }
    }
}
__device__ __forceinline__ void power_rows(const Power &a, int64_t which, int64_t r0, int64_t d, int64_t cols, int64_t ld,
                                           const double *__restrict__ y, double *__restrict__ z, double *vec) {
    static_assert(kSquareLeast > 2 * kWave, "fewer columns are not squared");
    if (cols <= 6 * kWave) power_rows<3, 8>(a, which, r0, d, cols, ld, y, z, vec);
    else power_rows<8, 4>(a, which, r0, d, cols, ld, y, z, vec);
}

// A square in blocks of 16 x 16 on and above the diagonal, which go in strips: the groups of columns 2 p and 2 p + 1 against four groups
// from 2 p + 4 q on (fewer at the end; the block below the diagonal in the first strip of a row is left out).
constexpr int kBlock = kGroup * kGroup, kTurns = 4;
static_assert(kBlock == kTileThreads, "an entry per thread");
// v_mfma_f64_4x4x4 forms four 4 x 4 products side by side: lane l gives row l / 16 of four and column l % 16 of a
// group, and quad b of the columns of the one operand meets quad b of the other.  So the one is also taken turned by one, two and three
// quads, and sum r of lane l is entry (4 ((l / 4 + r) % 4) + l % 4, 4 (l / 4 % 4) + l / 16) of the 16 x 16 product.  v_mfma_f64_16x16x4
// needs no turns, but takes 100 to 140 clocks for the work of four of these at 16: 45 TFLOP/s on the whole chip against 73.
// Vector instructions and these do not overlap, so what is turned serves four groups: with two 58 TFLOP/s are left, with four 67.
template <int CTRL>
__device__ __forceinline__ double turned(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// The strip whose first columns are ci and cj of M^T M, M [rows][ld] with rows a multiple of 16, by a workgroup, its four wavefronts four
// rows each of every sixteen: put(i, j, row, column, sum) for the entries of its blocks.  red: LDS.
template <int HIGH, int WIDE, bool DIAGONAL, class Put>
__device__ __forceinline__ void square_strip(const double *__restrict__ M, int32_t rows, int64_t ld, int32_t ci, int32_t cj,
                                             double (*red)[kWide][kBlock], Put put) {
    constexpr int kInFlight = 2;                     // steps per buffer
    const int wave = threadIdx.x / kWave, lane = lane_id();
    const int64_t step = (int64_t)kTileWaves * kStepRows * ld;
    const double *from_i = M + (wave * kStepRows + lane / 16) * ld + ci + (lane & 15), *from_j = from_i + (cj - ci);
    double e[HIGH][WIDE][kTurns] = {};
    struct Step {
        double i[HIGH], j[WIDE];
    };
    auto load = [&](int32_t at, Step &v) {
#pragma unroll
        for (int t = 0; t < HIGH; ++t) v.i[t] = from_i[at * step + t * kGroup];
#pragma unroll
        for (int t = 0; t < WIDE; ++t) v.j[t] = from_j[at * step + t * kGroup];
    };
    auto multiply = [&](const Step &v) {
#pragma unroll
        for (int i = 0; i < HIGH; ++i) {
            const double a[kTurns] = {v.i[i], turned<0x12c>(v.i[i]), turned<0x128>(v.i[i]), turned<0x124>(v.i[i])};   // row_ror by 12, 8, 4
#pragma unroll
            for (int r = 0; r < kTurns; ++r)
#pragma unroll
                for (int j = DIAGONAL ? i : 0; j < WIDE; ++j) e[i][j][r] = __builtin_amdgcn_mfma_f64_4x4x4f64(v.j[j], a[r], e[i][j][r], 0, 0, 0);
        }
    };
    // two buffers in turn: the one's loads are in flight while the other is multiplied; a step past the end loads the last one
    const int32_t steps = rows / (kTileWaves * kStepRows), last = steps - 1;
    Step v[kInFlight], w[kInFlight];
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) load(u < last ? u : last, v[u]);
    for (int32_t at = 0; at < steps; at += 2 * kInFlight) {
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) load(at + kInFlight + u < last ? at + kInFlight + u : last, w[u]);
#pragma unroll
        for (int u = 0; u < kInFlight; ++u)
            if (at + u < steps) multiply(v[u]);
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) load(at + 2 * kInFlight + u < last ? at + 2 * kInFlight + u : last, v[u]);
#pragma unroll
        for (int u = 0; u < kInFlight; ++u)
            if (at + kInFlight + u < steps) multiply(w[u]);
    }
    const int t = threadIdx.x, quad = (lane >> 2) & 3, row = 4 * ((quad + wave) & 3) + (lane & 3), col = 4 * quad + (lane >> 4);
#pragma unroll
    for (int i = 0; i < HIGH; ++i) {
        const int j0 = DIAGONAL ? i : 0;
        if (i > 0) __syncthreads();                  // what was there before has been read
#pragma unroll
        for (int j = j0; j < WIDE; ++j)
#pragma unroll
            for (int r = 0; r < kTurns; ++r) red[wave][j][r * kWave + lane] = e[i][j][r];
        __syncthreads();
        for (int j = j0; j < WIDE; ++j)              // this wavefront's entries are those of turn `wave`
            put(i, j, row, col, ((red[0][j][t] + red[1][j][t]) + red[2][j][t]) + red[3][j][t]);
    }
}
static_assert(kTurns == kTileWaves, "see square_strip");

// to = M M (both scaled as above; to's traces in an entry per row of strips), a workgroup per strip, consecutive ones
// on one XCD; and, by the workgroups beyond, z = M y where z is given: M stands for G^(2^j), and the exponent asked for has that bit.
// Bound by the matrix cores, three workgroups to a compute unit, and by there being two or three of them: 21 matrices of d = 300 are
// 630 strips for 256 units, 24.5 us where the products take 11.
__global__ __launch_bounds__(kTileThreads, 3) void gram_square_kernel(Power a, int64_t d, int64_t ld, int32_t groups, int32_t strips,
                                                                      int32_t matrices, double *__restrict__ to,
                                                                      double *__restrict__ to_traces, const double *__restrict__ y,
                                                                      double *__restrict__ z) {
    __shared__ double red[kTileWaves][kWide][kBlock];
    const int32_t cols = groups * kGroup, units = matrices * strips, per = (units + (int32_t)kXcds - 1) / (int32_t)kXcds;
    if ((int32_t)blockIdx.x >= per * (int32_t)kXcds) {               // rows of M y
        const int32_t at = (int32_t)blockIdx.x - per * (int32_t)kXcds, blocks = (int32_t)ld / kMvRows;
        power_rows(a, at / blocks, at % blocks * kMvRows, d, cols, ld, y, z, &red[0][0][0]);
        return;
    }
    const int32_t unit = (int32_t)blockIdx.x % (int32_t)kXcds * per + (int32_t)blockIdx.x / (int32_t)kXcds;
    if (unit >= units) return;
    const int32_t which = unit / strips;
    const double part = trace_part(a, which);
    int32_t p = 0, q = unit % strips;
    for (int32_t here; q >= (here = (groups - 2 * p + kWide - 1) / kWide); ++p) q -= here;
    double *out = to + which * ld * ld, diagonal = 0.0, scale = 0.0;
    auto put = [&](int i, int j, int r, int c, double sum) {
        if (scale == 0.0) {
            scale = unit_scale(part);
            scale *= scale;
        }
        const int32_t gi = 2 * p + i, gj = 2 * p + kWide * q + j;
        const int64_t row = gi * kGroup + r, col = gj * kGroup + c;
        sum *= scale;
        out[row * ld + col] = sum;
        if (gi != gj) out[col * ld + row] = sum;
        else if (r == c) diagonal += sum;
    };
    const double *M = a.M + which * ld * ld;
    const int32_t ci = 2 * p * kGroup, cj = ci + kWide * q * kGroup, left = groups - 2 * p - kWide * q;
    if (q == 0) {
        if (left == 1) square_strip<1, 1, true>(M, cols, ld, ci, cj, red, put);
        else if (left == 2) square_strip<2, 2, true>(M, cols, ld, ci, cj, red, put);
        else if (left == 3) square_strip<2, 3, true>(M, cols, ld, ci, cj, red, put);
        else square_strip<2, 4, true>(M, cols, ld, ci, cj, red, put);
    } else {
        if (left == 1) square_strip<2, 1, false>(M, cols, ld, ci, cj, red, put);
        else if (left == 2) square_strip<2, 2, false>(M, cols, ld, ci, cj, red, put);
        else if (left == 3) square_strip<2, 3, false>(M, cols, ld, ci, cj, red, put);
        else square_strip<2, 4, false>(M, cols, ld, ci, cj, red, put);
    }
    if (q > 0) return;
    diagonal = wave_sum_f64(diagonal);
    __syncthreads();
    if (lane_id() == 0) red[0][0][threadIdx.x / kWave] = diagonal;
    __syncthreads();
    if (threadIdx.x == 0) to_traces[which * kTraces + p] = (red[0][0][0] + red[0][0][1]) + (red[0][0][2] + red[0][0][3]);
}

__global__ __launch_bounds__(kMvThreads) void gram_apply_kernel(Power a, int64_t d, int64_t cols, int64_t ld, const double *__restrict__ y,
                                                                double *__restrict__ z) {
    __shared__ double vec[kGramMax];
    power_rows(a, blockIdx.y, (int64_t)blockIdx.x * kMvRows, d, cols, ld, y, z, vec);
}

// stats[row] = (0, |z| / |y|), z the product of y and G scaled and lifted as above.
__global__ __launch_bounds__(kMvThreads) void gram_ratio_kernel(Power a, const double *__restrict__ y, const double *__restrict__ z,
                                                                int64_t ld, double2 *__restrict__ stats) {
    __shared__ double sums[2][kMvWaves];
    constexpr int kPer = (int)kGramMax / kMvThreads;
    const int64_t which = blockIdx.x;
    const double part = trace_part(a, which);
    double vy[kPer], vz[kPer], sy = 0.0, sz = 0.0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int64_t j = threadIdx.x + q * kMvThreads;
        vy[q] = j < ld ? y[which * ld + j] : 0.0;
        vz[q] = j < ld ? z[which * ld + j] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        sy += vy[q] * vy[q];
        sz += vz[q] * vz[q];
    }
    sy = wave_sum_f64(sy);
    sz = wave_sum_f64(sz);
    if (lane_id() == 0) {
        sums[0][threadIdx.x / kWave] = sy;
        sums[1][threadIdx.x / kWave] = sz;
    }
    const double scale = a.lift * unit_scale(part);
    __syncthreads();
    if (threadIdx.x > 0) return;
    sy = (sums[0][0] + sums[0][1]) + (sums[0][2] + sums[0][3]);
    sz = (sums[1][0] + sums[1][1]) + (sums[1][2] + sums[1][3]);
    static_assert(kMvWaves == 4, "four sums");
    stats[which] = make_double2(0.0, sqrt(sz) * inverse_norm(sy) / scale);
}

template <int NC>
void launch_resident(const GramWs &ws, int32_t n, int64_t d, int64_t ld, int32_t iterations, double *stats, hipStream_t stream) {
    if (const int32_t steps = lanczos_steps(iterations)) {
        hipLaunchKernelGGL((gram_resident_kernel<NC, true>), dim3((unsigned)(n + 1)), dim3(kResThreads), 0, stream, ws.G, d, ld,
                           iterations, steps, true, ws.v, (double2 *)stats);
        return;
    }
    for (int32_t done = 0; done < iterations; done += kItersPerLaunch) {
        const int32_t now = iterations - done < kItersPerLaunch ? iterations - done : kItersPerLaunch;
        hipLaunchKernelGGL((gram_resident_kernel<NC, false>), dim3((unsigned)(n + 1)), dim3(kResThreads), 0, stream, ws.G, d, ld,
                           now, 0, done == 0, ws.v, (double2 *)stats);
    }
}

}  // namespace

hipError_t launch_gram_power(const float *A, int32_t n, int64_t m, int64_t d, int32_t iterations, int32_t squarings, void *workspace,
                             double *stats, hipStream_t stream) {
    const GramPlan p = gram_plan(n, m, d);
    if (d > kGramMax || p.chunks > 65535 || n > 65534 || (squarings >= 0 && d < kSquareLeast)) return hipErrorInvalidValue;
    GramWs ws;
    gram_layout(n, p, squarings >= 0, (char *)workspace, &ws);
    const int64_t units = n * p.chunks;
    hipLaunchKernelGGL(gram_tile_kernel, dim3((unsigned)((units + kXcds - 1) / kXcds * kXcds * p.pairs)), dim3(kTileThreads),
                       0, stream, A, m, d, p.rows_per_chunk, p.chunks, units, p.pairs, ws.part);
    const dim3 finish_grid((unsigned)p.pairs, (unsigned)(n + 1));
    if (squarings >= 0) {
        hipLaunchKernelGGL(gram_finish_kernel<double>, finish_grid, dim3(kTileThreads), 0, stream, ws.part, p.chunks, p.pairs,
                           d, p.ld, (double)m, ws.power[0], ws.traces[0]);
        const double lift = std::exp2(std::ceil(0.5 * std::log2((double)d)));
        const Power G{ws.power[0], ws.traces[0], (int32_t)p.nb, lift};
        Power now = G;
        const double *y = nullptr;                   // the start vector
        double *z = ws.v, *other = ws.w;
        auto applied = [&]() {
            y = z;
            std::swap(z, other);
        };
        const int64_t groups = (d + kGroup - 1) / kGroup, strips = strip_count(groups), row_blocks = p.ld / kMvRows;
        const int32_t rest = iterations - 1;
        for (int32_t j = 0; j < squarings; ++j) {
            const int to = 1 + j % 2;
            const bool apply = (rest >> j) & 1;
            const int64_t grid = ((n + 1) * strips + kXcds - 1) / kXcds * kXcds + (apply ? (n + 1) * row_blocks : 0);
            hipLaunchKernelGGL(gram_square_kernel, dim3((unsigned)grid), dim3(kTileThreads), 0, stream, now, d, p.ld, (int32_t)groups,
                               (int32_t)strips, n + 1, ws.power[to], ws.traces[to], y, z);
            if (apply) applied();
            now = Power{ws.power[to], ws.traces[to], (int32_t)((groups + 1) / 2), lift};
        }
        const dim3 apply_grid((unsigned)row_blocks, (unsigned)(n + 1));
        for (int32_t i = 0; i < rest >> squarings; ++i) {
            hipLaunchKernelGGL(gram_apply_kernel, apply_grid, dim3(kMvThreads), 0, stream, now, d, groups * kGroup, p.ld, y, z);
            applied();
        }
        hipLaunchKernelGGL(gram_apply_kernel, apply_grid, dim3(kMvThreads), 0, stream, G, d, groups * kGroup, p.ld, y, z);
        hipLaunchKernelGGL(gram_ratio_kernel, dim3((unsigned)(n + 1)), dim3(kMvThreads), 0, stream, G, y, z, p.ld, (double2 *)stats);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(gram_finish_kernel<float>, finish_grid, dim3(kTileThreads), 0, stream, ws.part, p.chunks, p.pairs, d,
                       p.ld, (double)m, ws.G, (double *)nullptr);
    if (d <= kResidentMax) {
        switch ((d + kWave - 1) / kWave) {
            case 1: launch_resident<1>(ws, n, d, p.ld, iterations, stats, stream); break;
            case 2: launch_resident<2>(ws, n, d, p.ld, iterations, stats, stream); break;
            case 3: launch_resident<3>(ws, n, d, p.ld, iterations, stats, stream); break;
            case 4: launch_resident<4>(ws, n, d, p.ld, iterations, stats, stream); break;
            default: launch_resident<5>(ws, n, d, p.ld, iterations, stats, stream); break;
        }
        return hipGetLastError();
    }
    hipLaunchKernelGGL(gram_start_kernel, dim3((unsigned)((p.ld + kTileThreads - 1) / kTileThreads), (unsigned)(n + 1)),
                       dim3(kTileThreads), 0, stream, ws.v, d, p.ld);
    double *from = ws.v, *to = ws.w;
    const dim3 grid((unsigned)(p.ld / kMvRows), (unsigned)(n + 1));
    if (const int32_t steps = lanczos_steps(iterations)) {
        const size_t vector = (size_t)(n + 1) * p.ld;
        double *v3[3] = {ws.lanczos, ws.lanczos + vector, ws.lanczos + 2 * vector};
        double *alpha = ws.lanczos + 3 * vector, *beta = alpha + (size_t)(n + 1) * kLanczosMax;
        for (int32_t j = 0; j < steps; ++j) {       // launch j: v_{j+1}, in v3[(j + 1) % 3], and its product
            const Recurrence r{j, v3[j % 3], v3[(j + 2) % 3], v3[(j + 1) % 3], alpha, beta};
            hipLaunchKernelGGL(gram_matvec_kernel, grid, dim3(kMvThreads), 0, stream, ws.G, p.ld, from, to, r);
            std::swap(from, to);
        }
        hipLaunchKernelGGL(gram_tridiagonal_kernel, dim3((unsigned)(n + 1)), dim3(kWave), 0, stream, from, v3[steps % 3], p.ld,
                           alpha, beta, steps, iterations, (double2 *)stats);
        return hipGetLastError();
    }
    for (int32_t it = 0; it < iterations; ++it) {
        hipLaunchKernelGGL(gram_matvec_kernel, grid, dim3(kMvThreads), 0, stream, ws.G, p.ld, from, to,
                           Recurrence{-1, nullptr, nullptr, nullptr, nullptr, nullptr});
        std::swap(from, to);
    }
    hipLaunchKernelGGL(gram_norm_kernel, dim3((unsigned)(n + 1)), dim3(kWave), 0, stream, from, p.ld, (double2 *)stats);
    return hipGetLastError();
}

}  // namespace ef21
