// What the host decides about a clip search (Algorithm 1, section 4.1): how many steps it can take, how batches of clip ratios
// cover them, and whether the grid form (kernels_gridsearch.hip) is the faster one.  Plain host code.
#pragma once
#include <algorithm>
#include <cstdint>

namespace rq {

// Steps a batch of the search looks ahead: up to 5 (the 31 nodes of the outcome tree, plus the starting point in the
// first batch) on small tensors, up to 3 (7 nodes + 1) on large ones, where the extra candidates would cost more than
// the passes they save.
constexpr int64_t kGbsSmall = (int64_t)1 << 22;              // rows * n up to which 5 steps are taken
inline int gbs_depth(int64_t rows, int n) { return (double)rows * (double)n <= (double)kGbsSmall ? 5 : 3; }

// Most steps a search down to a bracket of eps can take: two steps halve the bracket (from 1, by way of 3/4).  That
// holds while the midpoints are exact; a bracket of a few ulps stops shrinking and the search goes on to its limit.
inline int gbs_most_steps(double eps, int limit) {
    if (eps < 0x1p-50) return limit;
    int steps = 0;
    for (double w = 1.0; w > eps && steps < limit; ++steps) w = steps % 2 == 0 ? w * 0.75 : w / 1.5;
    return steps;
}

// As few batches as the depth allows, each no deeper than that number needs (16 steps: four batches of four, 61
// candidates, where batches of five would evaluate 95).
struct GbsBatches { int count, depth; };
inline GbsBatches gbs_batches(int64_t rows, int n, int steps) {
    if (steps < 1) return GbsBatches{1, 1};
    const int deepest = gbs_depth(rows, n), count = (steps + deepest - 1) / deepest;
    return GbsBatches{count, (steps + count - 1) / count};
}
constexpr int kStepsAhead = 3;                               // steps of a search that a step of the resident form decides

// Clip ratios m / kGridRatios of the grid form, and the 64-bit words of LDS that a row's histogram takes (error_grid.h).
constexpr int kGridRatios = 512, kGridGroups = 256;          // (and the most workgroups that take part)
constexpr int grid_cells(int bits) { return (2 * ((1 << (bits - 1)) - 1) - 1) * (kGridRatios - 1) + 1; }
constexpr int grid_words(int bits) { return grid_cells(bits) + kGridRatios; }
constexpr int kGridSpread = 16;                              // words that share the last cell of either histogram
// Rows whose histograms a workgroup can hold side by side: two, one, or none where not even one fits beside `other` bytes of
// LDS and a margin for what the kernels keep in static arrays (448 bytes, 640 with several rows a pass) and the histograms' further
// words (up to 320 bytes a row, 288 with two rows); the kernels hold themselves to it.
constexpr int kGridMargin = 1024;
constexpr int grid_rows_beside(int bits, int64_t max_lds, int64_t other = 0) {
    const int64_t row = 8 * (int64_t)grid_words(bits), left = max_lds - other - kGridMargin;
    return left >= 2 * row ? 2 : left >= row ? 1 : 0;
}

struct GridCase {
    int64_t rows;
    int n, bits, cus;
    bool sylvester;
    int beside;             // rows that fit a workgroup's LDS, see above
    int waves;              // a row's in the resident form; 0: a row of the workgroup block kernel, for which
    int rows_per_pass;      // are its own rows per pass
    int threads;            // and threads
};

// Whether the grid form is the faster one for a search of up to `steps` steps: its time does not depend on them, that of the
// forms it competes with (resident where the chip holds the tensor, else batches) grows with them.  Straight lines through
// 4400 pairs of measured times, us (25 orders from 384 to 32768, 1 to 32768 rows, 0 to 16 steps, both code widths), of a grid form
// up to 25 % slower than the present one, so that the border leans to the other forms: of 8064 pairs measured with the present one (the same
// orders, 14 row counts, 12 numbers of steps, normal rows) the form taken is within a tenth of the faster one but for 236, of
// which 16 are grid; at worst it is 1.34 times it (32768 x 28672, b = 4, four steps, 2285 and 1710; 1536 x 256, b = 4, six, 25.2 and 19.3).
// 4096 x 2048 rows, b = 3: grid 39 - 40 at any number of steps; batches 26 for up to two, 33 for three, 54 for five, 135 for sixteen.
// 1024 x 8192 rows: 86 - 88; 28, 32, 53, 132.  4096 x 64 rows: 17 - 19; resident 13, 13, 17, 33.  18944 x 512 rows: 31 - 33; 29, 35, 59, 149.
inline bool gbs_grid_pays(const GridCase& c, int steps) {
    if (c.beside < 1) return false;
    const double kilo = c.n / 1024.0, load = (double)c.rows * c.n / (4096.0 * c.cus);     // 4096 values a compute unit
    const GbsBatches b = gbs_batches(c.rows, c.n, steps);
    const int fours = ((1 << b.depth) + 3) / 4;              // clip ratios of a batch are taken four at a time
    if (c.waves > 0) {
        // a pass of the grid form: two rows a compute unit, or one where that is all there is
        const double row = (c.bits == 3 ? 4.4 : 5.7) + 0.95 * kilo + (c.sylvester ? 0.0 : 0.7);
        const int64_t two = 2 * (int64_t)c.cus;
        const double grid = 14.5 + (c.rows <= c.cus ? 0.5 * row : (double)((c.rows + two - 1) / two) * row * (c.beside > 1 ? 1.0 : 2.0));
        if (c.rows <= (int64_t)c.cus * (16 / c.waves))
            return grid < 9.0 + std::max(1, (steps + kStepsAhead - 1) / kStepsAhead) * (4.0 + 1.3 * load);
        return grid < 14.0 + b.count * (9.5 + load * (0.2 + 0.6 * fours));
    }
    // the rows of a pass share one histogram: one row after the other
    const int64_t passes = (c.rows + c.rows_per_pass - 1) / c.rows_per_pass;
    const int64_t serial = std::min<int64_t>(c.rows, c.rows_per_pass * ((passes + c.cus - 1) / c.cus));
    const double row = (c.rows_per_pass > 1 ? 5.0 : 2.25) + 0.12 * grid_words(c.bits) / c.threads + 0.47 * kilo;
    return 15.0 + serial * row < 8.0 + b.count * (13.0 + 0.5 * fours + load * (0.55 + 0.58 * fours));
}

}  // namespace rq
