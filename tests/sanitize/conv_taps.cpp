// Host walk over the rows of a chunk as the fetching threads of a wide-tile convolution take them by tap (csrc/conv_taps.hpp).
#include <cstddef>
#include <vector>

#include "conv_taps.hpp"

// -1: rows are not dealt by tap; otherwise how many (row, piece) units of a chunk are not fetched exactly once, for every tap that
// the chunk's first row can be
extern "C" int conv_tap_faults(int tn, int KK, int chunk_rows) {
    const int ways = grim::conv_tap_ways(tn, KK, chunk_rows), pieces = tn / 8, pairs = KK * pieces;
    if (ways == 0) return -1;
    int bad = 0;
    for (int first = 0; first < KK; ++first) {
        std::vector<int> met((std::size_t)chunk_rows * pieces, 0);
        for (int thread = 0; thread < grim::kWideFetchThreads; ++thread) {
            const int way = thread / pairs, pair = thread - way * pairs, tap = pair / pieces, c = pair - tap * pieces;
            if (way >= ways) continue;
            for (int i = 0; i < grim::wide_tap_units(tn); ++i) {
                const int row = (way + i * ways) * KK + tap - first + (tap < first ? KK : 0);
                if (row < chunk_rows) ++met[(std::size_t)row * pieces + c];
            }
        }
        for (int n : met) bad += n != 1;
    }
    return bad;
}
