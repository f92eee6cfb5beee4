// Rules of the sequence kernel that the host can check: which sets of workgroups run on an XCD of their own and how, and when a
// thread's waits end.
#pragma once
#include <cstdint>

#include "host_device.hpp"

namespace grim {

// A set's workgroups on one XCD (workgroup ids are dealt to the eight of them round-robin): the exchange words of a set are
// then written and read from there alone.  Workgroups of a call wait for one another, so all of them have to be resident:
// only calls whose sets come in multiples of eight are placed so, because these put as many workgroups on every XCD as the
// plain order does.  Placing fewer sets would crowd calls that overlap on several streams onto the same few XCDs, where each
// could hold a part of the compute units and wait for the rest.
GRIM_HOST_DEVICE bool seq_sets_on_xcds(int sets) { return sets % 8 == 0; }

// set and number inside the set of workgroup `id` of a 1-D grid of sets * wgs workgroups
GRIM_HOST_DEVICE void seq_placed_at(int id, int wgs, int *set, int *unit) {
    const int slot = id >> 3;
    *set = slot / wgs * 8 + (id & 7);
    *unit = slot % wgs;
}

// Forms of a call: sets in grid.y, placed as above, or claimed by the XCDs (bcr_rnn_seq.hip).  Claimed are sets of workgroups that an
// XCD's 32 compute units hold one each of, in sequences long enough to pay for the claim (2 us; a step on one XCD is 0.4 to 0.5 us
// shorter than one across them: an LSTM of 1024 / 512 / 256 units, one sequence of 64 steps 132 / 129 / 130 -> 107 / 104 / 96 us, GRU
// 137 / 139 / 149 -> 114 / 109 / 104, four sequences of 1024 units 135 -> 109, 137 -> 116).
constexpr int kSeqPlain = 0, kSeqPlaced = 1, kSeqClaimed = 2;
GRIM_HOST_DEVICE bool seq_sets_claimed(int sets, int64_t wgs, int steps) {
    return sets % 8 != 0 && wgs > 1 && (sets + 7) / 8 * wgs <= 32 && steps >= 8;
}

// A step's waits of one thread, `per_wait` of the `pairs` of its workgroup's sequences at a time: once one has been given up (false)
// no further one begins, so that a thread gives up after its limit of reads however many sequences its workgroup carries.
template <class Wait>
GRIM_HOST_DEVICE bool seq_waits(int pairs, int per_wait, Wait wait) {
    for (int q0 = 0; q0 < pairs; q0 += per_wait)
        if (!wait(q0)) return false;
    return true;
}

}  // namespace grim
