// Host side of the block-scaled kernels (itq3s_mx.hip, itq3s_gemm.hip): the layout of their operand, what scratch it
// takes, and which kernel computes a call with more than 16 rows.  Plain C++, no HIP.
#pragma once
#include <cstddef>
#include <cstdint>

#include "itq3s_rows_rule.h"

namespace itq3s {

// 32 activation rows of a 256-channel block together: four steps of 64 channels, each three parts of 64 lanes x (16 + 8)
// bytes, then what belongs to the block: the lanes' scales (a byte a step), 32 times -S, 32 times E.
constexpr int kMxRows = 32;
constexpr int kMxPartBytes = 1536;
constexpr int kMxStepBytes = 3 * kMxPartBytes;             // 4608
constexpr int kMxMetaBytes = 64 * 4 + 32 * 4 + 32 * 4;     // 512
constexpr int kMxBlockBytes = 4 * kMxStepBytes + kMxMetaBytes;  // 18944
inline size_t mx_bytes(int64_t M, int64_t K) { return (size_t)((M + kMxRows - 1) / kMxRows) * (size_t)(K / 256) * kMxBlockBytes; }

constexpr int kMxWaves = 8;  // wavefronts of a workgroup of mx_kernel
enum class Route { rows, shares8, shares4, tiled };

// Times of a call in us, the rotation in front among it: fits to 269 sizes (24 to 2048 rows, 512 to 28672 columns, K 1024 to
// 28672, 256 units; root mean square of the relative error 0.05, 0.07, 0.07 for 32, 64 and 128 columns an item, 0.04 for
// the other two).  mx_kernel: rounds of items of 32 rows by 32 nt (shares8) or 256 columns (shares4); a round costs
// its end and its steps, both more the fuller it is.
inline double shares_time(const double (&c)[6], int64_t items, int64_t steps, int64_t M, int64_t K, int units) {
    const double rounds = (double)((items + units - 1) / units), full = (double)items / units;  // (rounds x how full they are)
    return c[0] + rounds * c[1] + full * c[2] + (double)steps * (rounds * c[3] + full * c[4]) + c[5] * 1e-6 * (double)M * (double)K;
}
inline double shares8_time(int64_t col_tiles, int nt, int64_t M, int64_t K, int units) {
    constexpr double c[3][6] = {{7.81, -0.51, 1.11, 1.84, 0.0, 1.47}, {7.89, -0.23, 1.07, 2.02, 0.11, 1.21}, {8.7, 0.03, 1.24, 2.51, 0.5, 1.02}};
    return shares_time(c[nt == 1 ? 0 : nt == 2 ? 1 : 2], (M + kMxRows - 1) / kMxRows * col_tiles, (K / 256 + 7) / 8, M, K, units);
}
// Columns of an item over 32 for a launch of these tensors: what takes the fewest rounds' time for the launch as a whole (a
// column's sums do not depend on it).
inline int shares8_columns(const int64_t* N, int count, int64_t M, int64_t K, int units) {
    int best_nt = 1;
    double best = 1e300;
    for (int nt = 1; nt <= 4; nt *= 2) {
        int64_t cols = 0;
        for (int i = 0; i < count; ++i) cols += (N[i] + 32 * nt - 1) / (32 * nt);
        const double t = shares8_time(cols, nt, M, K, units);
        if (t < best) { best = t; best_nt = nt; }
    }
    return best_nt;
}
inline double shares4_time(int64_t M, int64_t N, int64_t K, int units) {
    constexpr double c[6] = {9.13, 1.1, 1.74, 2.22, 0.51, 0.86};
    return shares_time(c, (M + kMxRows - 1) / kMxRows * ((N + 255) / 256), (K / 256 + 3) / 4, M, K, units);
}
// gemm_kernel: tiles of 64 x 256, two to a unit.
inline double tiled_time(int64_t M, int64_t N, int64_t K, int units) {
    const int64_t items = (M + 63) / 64 * ((N + 255) / 256), most = (items + units - 1) / units;
    const double per_block = (most == 1 ? 1.51 : 0.88) + 1.385 * (double)(most - 1) + 0.226 * (double)items / units;
    return 9.5 + per_block * (double)(K / 256) + 1e-6 * (double)M * (double)K;
}
// The many-row kernel (its cost counts rounds and steps; with one step a round's end hides behind the next).
inline double rows_time(int64_t M, int64_t N, int64_t K, int units) {
    const RowsSplit s = rows_split((N + 15) / 16, M, K, units);
    const double mk = 1e-6 * (double)M * (double)K;
    if (K <= 2048) return 6.3 + (double)s.cost / 64.7 + 1.68 * mk - 4.07 * (double)s.rounds;
    return 3.0 + (double)s.cost / 67.3 + 2.0 * mk;
}

// Which kernel computes a tensor (M >= 17): among the block-scaled ones the fastest by the times above; the many-row kernel,
// where its own rule takes the call,
//  - below a line of rows (480, with K beyond 8192 fewer: 70 at 28672) or of 1.6 million activations, unless they save what
//    a tensor an eighth as wide takes by itself, less its share of a joint launch: that is k or v beside q with grouped
//    queries (8192 + 1024 + 1024 columns).  The tensors of a group go each by this rule, and a thin one left behind costs a
//    rotation and a launch with all of K.  us, one launch of the many-row kernel / q here and k, v there by the faster
//    kernel alone: K = 8192, 8192 + 1024 + 1024, M = 32 18.8 / 27.8, 48 22.1 / 32.6, 64 24.8 / 32.5, 100 40.6 / 40.0, 149 53.0 / 47.3, 300
//    80.6 / 66.7; K = 4096, 4096 + 1024 + 1024, M = 100 16.6 / 24.6, 149 22.2 / 28.7, 256 25.1 / 33.4, 300 30.5 / 34.6, 400 44.0 / 35.1.  A tensor
//    without such a sibling pays for it: 11008x4090, M = 149 30.6 / 27.3, 256 35.6 / 30.1; 8192x8192, M = 100 27.5 / 23.7.
//  - above it, not at all, whatever the columns: from 1024 on the block-scaled kernels are the faster ones there (0.71 to
//    1.0 of the time), and thinner tensors lose up to 5 % (512 columns, K = 8192, M = 366 21.1 / 22.2), 64 to 264 up to 10 %.
// A rule on the sizes of one tensor (counted for 256 units), and how a kernel adds up depends on K alone: a grouped call
// computes every tensor as a call of its own does.
inline Route many_row_route(int64_t M, int64_t N, int64_t K) {
    double best = shares8_time((N + 31) / 32, 1, M, K, 256);
    for (int nt = 2; nt <= 4; nt *= 2) {
        const double t = shares8_time((N + 32 * nt - 1) / (32 * nt), nt, M, K, 256);
        if (t < best) best = t;
    }
    Route route = Route::shares8;
    const double t4 = shares4_time(M, N, K, 256), tt = tiled_time(M, N, K, 256);
    if (t4 < best) { best = t4; route = Route::shares4; }
    // (tensors of a launch fill the tiled kernel's rounds together: 11008x4096, 512 rows 51 against 48 us, two of them 80 against 88)
    if (0.92 * tt < best) { best = tt; route = Route::tiled; }
    const int64_t line = K <= 8200 ? 480 : 644 - K / 50;
    if (rows_path(M, N, K) && (M < line || M * K < 1600000)) {
        const double rows = rows_time(M, N, K, 256);
        if (rows - best < rows_time(M, (N + 7) / 8, K, 256) - 0.1 * rows) return Route::rows;
    }
    return route;
}

}  // namespace itq3s
