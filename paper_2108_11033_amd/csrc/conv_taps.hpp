// How a wide-tile convolution's rows of a chunk are dealt to the fetching threads by kernel tap (kConvByTap of
// spmm_wide_kernel.hpp), shared with the host check that walks them.
#pragma once

namespace grim {

constexpr int kWideFetchWaves = 4;   // fetching waves
constexpr int kWideFetchThreads = kWideFetchWaves * 64;

// rows of a chunk a thread has registers for
constexpr int wide_tap_units(int tn) { return tn == 96 ? 11 : 15; }

// Fetching threads per (tap, piece of a tile of tn columns); 0: rows are not dealt by tap.  Not on 32-column tiles, a rest of a few
// workgroups whose chain of chunk periods is all there is to wait for: windows asked for one period ahead instead of two cost
// more there than the tables (with the rest by tap / from tables: 224 -> 352 channels, 3 x 3, on eleven 64 x 64 maps 143 / 118 us; 96 ->
// 448 on ten 104 x 40 82.6 / 71.8; 192 -> 352, 5 x 5, on six 56 x 104 236 / 215; 1 x 1, 512 -> 256 on five 112 x 112 39.3 / 36.6).
constexpr int conv_tap_ways(int tn, int KK, int chunk_rows) {
    const int pairs = KK * (tn / 8);
    const int ways = tn > 32 && pairs <= kWideFetchThreads ? kWideFetchThreads / pairs : 0;
    return ways > 0 && ((chunk_rows + KK - 1) / KK + ways - 1) / ways <= wide_tap_units(tn) ? ways : 0;
}

}  // namespace grim
