// Host walk over the workgroups of a sequence call (csrc/rnn_seq_placement.hpp): with `sets` sets of `wgs` workgroups, is
// every (set, unit) run by exactly one workgroup, and what is the largest number of workgroups an XCD receives -- against the
// plain order's, ids being dealt to the eight XCDs round-robin?
#include <algorithm>
#include <vector>

#include "rnn_seq_placement.hpp"

// < 0: not a permutation; else the XCD's load above the plain order's
extern "C" int seq_placement_excess(int sets, int wgs) {
    if (!grim::seq_sets_on_xcds(sets)) return 0;
    std::vector<int> seen((size_t)sets * wgs, 0), load(8, 0);
    for (int id = 0; id < sets * wgs; ++id) {
        int set = -1, unit = -1;
        grim::seq_placed_at(id, wgs, &set, &unit);
        if (set < 0 || set >= sets || unit < 0 || unit >= wgs || id % 8 != set % 8) return -1;
        if (seen[(size_t)set * wgs + unit]++) return -1;
        ++load[id % 8];
    }
    return *std::max_element(load.begin(), load.end()) - (sets * wgs + 7) / 8;
}
