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

extern "C" int seq_form_is_claimed(int sets, int wgs, int steps) { return grim::seq_sets_claimed(sets, wgs, steps); }

// reads a thread makes in a step of `pairs` pairs of sequences, `per_wait` at a time, whose wait number `fails` (< 0: none) never ends
// and is given up after max_polls of them
extern "C" int64_t seq_reads_of_a_step(int pairs, int per_wait, int fails, int max_polls) {
    int64_t reads = 0;
    const bool complete = grim::seq_waits(pairs, per_wait, [&](int q0) {
        const bool ends = fails < 0 || q0 / per_wait < fails;
        reads += ends ? 1 : max_polls;
        return ends;
    });
    return complete == (fails < 0) ? reads : -1;
}

// words by which the call with the most exchange words (of 1 .. 32 sequences through a layer of H units in strips of BR rows, on `cus`
// compute units) exceeds what a matrix of M rows has; <= 0: there is room
extern "C" int64_t seq_words_missing(int64_t M, int64_t H, int BR, int cus) {
    int64_t most = 0;
    for (int batch = 1; batch <= grim::kSeqMaxBatch; ++batch) {
        int sets, per_wg;
        grim::seq_split(H, BR, batch, cus, &sets, &per_wg);
        most = std::max(most, grim::seq_call_words(H, sets, per_wg) + grim::kSeqClaimWords);
    }
    return most - grim::seq_exchange_words(M);
}
