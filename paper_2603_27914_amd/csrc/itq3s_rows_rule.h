// Host side of the streaming kernel for many rows (itq3s_rows.hip): how a launch is divided, what scratch it
// takes, and which calls are its.  Plain C++, no HIP.
#pragma once
#include <cstddef>
#include <cstdint>

namespace itq3s {

constexpr int64_t kRowsMinM = 17;  // fewer rows: the streaming kernel of itq3s_gemv.hip
constexpr int64_t kRowsMaxM = 1 << 16;
constexpr int64_t kRowsMaxK = 1 << 18;
constexpr int kRowsWaves = 8;  // wavefronts per workgroup
constexpr int64_t kRowsMaxM1 = 96;  // groups of 16 rows up to here (beyond, their first elements could take more than rows_x0_bytes)
constexpr int kRowsMaxRT = 4;  // row tiles per item, at most (256 registers with 64 rows)

// Rows per group (16 mt) and row tiles per item (rt): the pair that takes the least time in rounds of one
// workgroup per compute unit (eight wavefronts of up to 256 registers).  An item costs per block of its
// wavefronts 23 for a row tile and 56 for 16 activation rows (their fragments' way through the L1), then 60 per
// row tile and 100 for its end: fitted to launches with every rt and mt (11008x4096, one round: 16.9 / 18.9 / 21.3 /
// 24.2 us for rt = 1..4 with mt = 2, 23.8 us for rt = 1, mt = 4).
struct RowsSplit {
    int mt, rt;
    int64_t items, rounds, cost;
};
inline RowsSplit rows_split(int64_t row_tiles, int64_t M, int64_t K, int units) {
    const int64_t steps = (K / 256 + kRowsWaves - 1) / kRowsWaves;
    RowsSplit best{2, 1, 0, 0, INT64_MAX};
    // Groups of 16 rows: thin tensors, which leave units idle otherwise (with all rows to a unit, all of the activations go through
    // each of the few units at 53 bytes a clock).  us without / with: 4096x1024 M = 48 8.6 / 7.1, 11008x512 M = 64 13.8 / 10.9,
    // 28672x1024 M = 24 33.3 / 22.5.  Not beyond what a chiplet's L2 holds (4 MB): 28672x1024 M = 64 33.8 / 24.3, M = 80 34.4 / 35.7.
    for (int m = M <= kRowsMaxM1 && M * K <= 2000000 ? 1 : 2; m <= 4; ++m) {
        const int64_t groups = (M + 16 * m - 1) / (16 * m);
        for (int r = 1; r <= kRowsMaxRT; ++r) {
            const int64_t items = (row_tiles + r - 1) / r * groups, rounds = (items + units - 1) / units;
            int64_t cost = rounds * (steps * (23 * r + 56 * m) + 60 * r + 100);
            if (m == 1) cost += cost / 10;  // (more items read the same weights: 28672x8192 M = 24, no fewer units without, 42.6 / 44.8)
            if (cost < best.cost) best = RowsSplit{m, r, items, rounds, cost};
        }
    }
    return best;
}

// Activation rows padded to whole groups of 32, 48 or 64: the most of the three (groups of 16 take no more).
inline int64_t rows_padded(int64_t M) {
    int64_t most = 0;
    for (int mt = 2; mt <= 4; ++mt) {
        const int64_t rows = (M + 16 * mt - 1) / (16 * mt) * (16 * mt);
        if (rows > most) most = rows;
    }
    return most;
}
inline size_t rows_xt_bytes(int64_t M, int64_t K) { return (size_t)rows_padded(M) * (size_t)K * 2; }
inline size_t rows_x0_bytes(int64_t M, int64_t K) { return (size_t)rows_padded(M) * (size_t)(K / 256) * 3; }  // 64 bytes per 16 or 32 rows, 128 per 48 or 64

// Which calls this kernel may take (many_row_route decides between it and the block-scaled ones, whose times are of the
// same form; where it may not, they take the call whatever their time).  Beyond 64 rows up to 36 GFLOP and 3.4 million
// outputs: there the block-scaled ones are ahead by a third (28672x8192 M = 96 83 / 50 us, K x N, here / there).  And not:
//  - short K: the ends of the items count, so a launch of more than so much cost (rows_split) loses against tiles.
//    Against tiles of fp16 operands: K = 256: cost 1719 16.3 / 16.6, 2400 20.2 / 16.1 (N = 28672, M = 65); K = 512: 2624
//    23.8 / 20.8; K = 1024: 2624 34.0 / 31.1; up to 64 rows 4800 39.7 / 40.5, 5248 48.5 / 41.5 (N = 128256, M = 56).
//  - more than 1280 rows: every round more reads the rotated activations through every chiplet's L2 again, which
//    does not hold them (N = 1000, K = 4096: M = 1024, one round, 24; 1500, two, 41; 2048, two, 52).
//  - 17 rows of a thin tensor with long K: two passes of the kernel for 16 rows, whose second rotates its one row
//    in the kernel, were 4 to 10 % faster than groups of 32 rows (N = 16, K = 28672 27.8 / 30.5).
// A rule on the sizes of one tensor (counted for 256 units): a grouped call computes every tensor as a call
// of its own does.
inline bool rows_path(int64_t M, int64_t N, int64_t K) {
    if (M < kRowsMinM || K > kRowsMaxK || M > kRowsMaxM) return false;
    // scratch: the padded rows must not take a call over a limit that rows as they are keep
    if (rows_xt_bytes(M, K) + rows_x0_bytes(M, K) > (32u << 20)) return false;
    if (M <= 32) return M > 17 || N > 1024 || K < 20480;
    if (M > 64 && ((double)M * (double)N * (double)K > 18e9 || (double)M * (double)N > 3.4e6)) return false;
    if (K >= 2048 && M <= 1280) return true;
    const RowsSplit s = rows_split((N + 15) / 16, M, K, 256);
    if (K < 2048) return s.cost <= (K <= 256 ? 1800 : K < 1024 ? 2400 : M > 64 ? 3000 : 4800);
    return s.rounds <= (K < 4096 ? 2 : 1);
}

}  // namespace itq3s
