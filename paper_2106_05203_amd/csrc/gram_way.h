// How the power iteration of a dense problem goes about it (gram_power.hip has the kernels): its workspace and which of the ways is taken.
// Plain C++ beside the kernels, so that the host can say for a shape which kernels a call of it reaches.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>

namespace ef21 {

constexpr int kTile = 32;                            // rows and columns of a tile of G
constexpr int kTileEntries = kTile * kTile;
constexpr int kGroup = 16, kWide = 4;                // a square's blocks, and how many of them lie side by side in a strip
constexpr int64_t kXcds = 8;                         // workgroups go round them one by one
constexpr int64_t kResidentWave = 64, kResidentMax = 5 * kResidentWave;   // columns (six would need 144 registers for G alone)
constexpr int64_t kGramMax = 1024;
constexpr int64_t kSquareLeast = 129;                // columns: see gram_way
constexpr int kTraces = 64;
constexpr size_t kGramWsMax = (size_t)1 << 30;

constexpr int kLanczosMax = 256;                     // steps of the recurrence: four per lane of the last wavefront
// Fewer iterations save next to nothing and a step takes longer than an iteration, us a call with the iteration and with the
// recurrence, 40 iterations (32 steps): n = 20, m = 1000, d = 64 71.3 and 72.7; 4, 250, 100 76.6 and 75.1; 16, 2000, 200 166.3
// and 166.4; 10, 3000, 500 520 and 455; 100 iterations (49 steps): 109 and 89, 131 and 96, 266 and 205, 960 and 580.
constexpr int32_t kLanczosLeast = 48;
// Steps that stand for `iterations` of the power iteration; 0: it is run as it is.
inline int32_t lanczos_steps(int32_t iterations) {
    if (iterations < kLanczosLeast) return 0;
    const int32_t steps = (int32_t)std::ceil(4.8 * std::sqrt((double)iterations)) + 1;
    return steps <= kLanczosMax ? steps : 0;
}

struct GramPlan {
    int64_t nb, pairs;              // tiles per side, tiles on and above the diagonal
    int64_t ld;                     // rows and row length of a padded G
    int64_t rows_per_chunk, chunks;
};

// Enough workgroups to fill the chip four deep, at least 256 rows (16 matrix instructions per wavefront and
// accumulator) each; up to three chunks more where that spreads the (worker, chunk) units evenly over the XCDs.
inline GramPlan gram_plan(int32_t n, int64_t m, int64_t d) {
    GramPlan p;
    p.nb = (d + kTile - 1) / kTile;
    p.pairs = p.nb * (p.nb + 1) / 2;
    p.ld = p.nb * kTile;
    int64_t chunks = 1024 / (n * p.pairs);
    if (chunks > m / 256) chunks = m / 256;
    if (chunks < 1) chunks = 1;
    const int64_t least = chunks;
    int64_t best = kXcds;
    for (int64_t c = least; c < least + 4 && (c == least || c <= m / 256); ++c) {
        const int64_t idle = (kXcds - n * c % kXcds) % kXcds;
        if (idle < best) {
            best = idle;
            chunks = c;
        }
    }
    p.rows_per_chunk = (m + chunks - 1) / chunks;
    p.chunks = (m + p.rows_per_chunk - 1) / p.rows_per_chunk;
    return p;
}

// A square's strips, see gram_square_kernel.
inline int64_t strip_count(int64_t groups) {
    int64_t strips = 0;
    for (int64_t p = 0; 2 * p < groups; ++p) strips += (groups - 2 * p + kWide - 1) / kWide;
    return strips;
}

struct GramWs {
    double *part;                   // [n][chunks][pairs][32][32]
    float *G;                       // [n + 1][ld][ld]
    double *v, *w;                  // [n + 1][ld] each
    double *lanczos;                // three more vectors of that size, and alpha and beta [n + 1][kLanczosMax]
    double *power[3];               // by squaring: G, and two matrices in turn, the first of them in part's place
    double *traces[3];              // [n + 1][kTraces] each
};

inline size_t gram_layout(int32_t n, const GramPlan &p, bool squaring, char *base, GramWs *ws) {
    size_t off = 0;
    // at whole 4096 bytes: the matrices' rows of d = 1000 otherwise straddle two channels' shares of memory (a product 13.4 us instead of 8.6)
    auto take = [&](size_t bytes) {
        char *at = base ? base + off : nullptr;
        off += (bytes + 4095) / 4096 * 4096;
        return at;
    };
    const size_t entries = (size_t)(n + 1) * p.ld * p.ld, part = sizeof(double) * (size_t)n * p.chunks * p.pairs * kTileEntries;
    GramWs out{};
    out.part = (double *)take(squaring ? std::max(part, sizeof(double) * entries) : part);
    if (squaring) {
        out.power[0] = (double *)take(sizeof(double) * entries);
        out.power[1] = out.part;
        out.power[2] = (double *)take(sizeof(double) * entries);
        for (auto &t : out.traces) t = (double *)take(sizeof(double) * (size_t)(n + 1) * kTraces);
    } else {
        out.G = (float *)take(sizeof(float) * entries);
        out.lanczos = (double *)take(sizeof(double) * (size_t)(n + 1) * (3 * p.ld + 2 * kLanczosMax));
    }
    out.v = (double *)take(sizeof(double) * (size_t)(n + 1) * p.ld);
    out.w = (double *)take(sizeof(double) * (size_t)(n + 1) * p.ld);
    if (ws) *ws = out;
    return off;
}

// bytes: of the workspace; 0: the iteration runs with A.  squarings: before the rest of the iterations is taken with the power reached
// (G^(2^s) applied (iterations - 1) >> s times, the other bits' powers beside the squarings), or -1: the iteration or the recurrence with G in fp32.
struct GramWay {
    size_t bytes = 0;
    int32_t squarings = -1;
};

// What follows are microseconds over what all ways on G have in common (forming it), from 2904 shapes of 129 to 1024 columns, 1 to 63 workers and
// eight numbers of iterations, each by every way.  Entries of all matrices, in millions.
inline double gram_entries(int32_t n, const GramPlan &p) { return 1e-6 * (n + 1.0) * (double)p.ld * (double)p.ld; }

// A squaring goes by the strips, 1.15 ns a step of sixteen rows (n = 3, d = 987 78; 20, 958 345; 62, 570 250); a product with a power by the last
// caches, which hold up to 4.4 million fp64 entries (n = 4, d = 568 5.2; 19, 649 11.7; 44, 793 35).
inline double squaring_us(int32_t n, const GramPlan &p, int64_t d, int32_t iterations, int32_t *squarings) {
    const int64_t groups = (d + kGroup - 1) / kGroup;
    const double entries = gram_entries(n, p), square = 9.0 + 1.15e-3 * (n + 1.0) * (double)(strip_count(groups) * groups);
    const bool cached = entries < 4.4;
    const double apply = cached ? 3.9 + 2.2e-3 * (double)d : 2.0 + 1.22 * entries, first = cached ? 0.0 : 2.0 * std::min(entries, 10.0);
    double least = 1e30;
    for (int32_t s = 0; s <= 20; ++s) {
        const double us = s * square + (double)(((iterations - 1) >> s) + 1) * apply + (s ? first : 0.0);
        if (us < least) {
            least = us;
            *squarings = s;
        }
    }
    return least;
}

// The recurrence, where it stands for the iterations, else the iteration, G in fp32.  Up to kResidentMax columns by wide = columns / 64 (us an
// iteration for three to five 1.2, 1.6 and 2.2, a step of the recurrence 2.2, 2.6 and 3.2, whose one launch has less to load); beyond, a launch a step
// of 6.2 to 8 while the last caches hold the matrices (a number of workgroups that is a multiple of the XCDs meets what the launch before left), then
// 9 (n = 41, d = 368) to 21 (44, 857), and a step of the recurrence 1.4 times that where there are more workgroups than fit at once.
inline double plain_us(int32_t n, const GramPlan &p, int64_t d, int32_t iterations) {
    const int32_t steps = lanczos_steps(iterations);
    if (d <= kResidentMax) {
        const double wide = (double)((d + kResidentWave - 1) / kResidentWave), turns = (double)((n + 256) / 256), sq = wide * wide;
        return steps ? 1.5 * sq - 36.0 + steps * turns * (1.55 + 0.068 * sq) : 1.25 * (sq - 5.0) + iterations * turns * (0.62 + 0.064 * sq);
    }
    const double entries = gram_entries(n, p);
    const int64_t blocks = (n + 1) * p.nb;
    const bool cached = entries < (blocks % kXcds == 0 ? 6.1 : 4.9);
    const double step = cached ? 5.4 + 2.8e-3 * (double)d : 4.5 + 7.5e-3 * (double)d + 0.28 * entries;
    if (steps) return steps * (step + 1.3) * (blocks > 1280 ? 1.4 : 1.0) - 12.0 - 0.9 * std::max(0.0, entries - 5.0);
    return iterations * step + (cached ? 8.0 : 3.0 - 1.8 * std::max(0.0, entries - 12.0));
}

// Squaring is taken where it is ahead by more than the formulas are off (five per cent and 3 us): of 23232 measured pairs 70 are then more than 3
// per cent slower than with G in fp32, 15 at most, and the mean is 0.6 per cent above the faster one of each pair.  A call of 100 iterations,
// us, by the recurrence and by squaring: n = 16, m = 2000, d = 200 204 and 179; 25, 800, 250 204 and 212; 20, 2487, 300 317 and 289; 32, 1400, 330
// 563 and 373; 10, 3000, 500 581 and 419; 3, 2000, 700 528 and 325; 2, 7500, 1000 796 and 656; 15, 1000, 1000 1154 and 1560; 1000 iterations of
// 20, 2487, 300 660 and 363; 20 of them 225 and 236.  Up to 128 columns the host's dozen launches are what counts: 4, 250, 100 95 and 101.
// squaring == false: without it, for a caller that has no memory for its workspace (six times the recurrence's per entry of G).
inline GramWay gram_way(int32_t n, int64_t m, int64_t d, int32_t iterations, bool squaring = true) {
    GramWay way;
    if (d > kGramMax || n > 65534) return way;
    const GramPlan p = gram_plan(n, m, d);
    const size_t plain = gram_layout(n, p, false, nullptr, nullptr), squared = gram_layout(n, p, true, nullptr, nullptr);
    int32_t squarings = -1;
    double with_g = 1e30;
    if (squaring && d >= kSquareLeast && iterations > 1 && squared <= kGramWsMax) {
        const double us = squaring_us(n, p, d, iterations, &squarings);
        if (1.05 * us + 3.0 < plain_us(n, p, d, iterations)) with_g = us;
        else squarings = -1;
    }
    if (squarings < 0 && plain > kGramWsMax) return way;
    // Microseconds, a handle's first call: forming the matrices (with the allocation of their workspace) and one iteration
    // on them (or one step of the recurrence), against one iteration with A (six launches).  Measured, forming | iteration on G | with A: n = 4, m = 250,
    // d = 100 1 | 0.9 | 22; 20, 2487, 300 172 | 2.5 | 44; 10, 3000, 500 223 | 7.3 | 40; 2, 7500, 1000 354 | 8.7 | 50;
    // 15, 1000, 1000 424 | 15 | 41; 32, 468, 1000 482 | 32 | 40; 32, 100, 1000 253 | 32 | 30; 1000, 20, 100 286 | 2.4 | 137.
    const double nn = n, mm = (double)m, dd = (double)d, ld = (double)p.ld, rows = nn * mm;
    const int32_t steps = lanczos_steps(iterations);
    const double step = d <= kResidentMax ? 2.6 * (double)((n + 256) / 256) : std::max(8.5, 0.92 * gram_entries(n, p));
    with_g = std::min(with_g, (steps ? steps : iterations) * step);
    const double form = 10.0 + 0.055 * dd + rows * ld * ld / 55e6 + 0.3e-6 * (double)plain;
    const double sums = 512.0 / nn < mm / 8.0 ? 512.0 / nn : mm / 8.0;           // of the gradient, per worker
    const double with_a = 22.0 + 1.1e-6 * rows * dd + 0.08 * nn + 3.5e-5 * sums * dd;
    if (form + with_g >= iterations * with_a) return way;
    way.squarings = squarings;
    way.bytes = squarings >= 0 ? squared : plain;
    return way;
}

}  // namespace ef21
