// Rules of the sequence kernel that the host can check: which sets of workgroups run on an XCD of their own and how, and when a
// thread's waits end.
#pragma once
#include <algorithm>
#include <cstdint>

#include "host_device.hpp"

namespace grim {

constexpr int64_t kSeqMaxH = 8192;
constexpr int32_t kSeqMaxBatch = 32;
constexpr int64_t kSeqClaimWords = 272;                            // words of a claim (seq_claim below) behind the exchange words

// `batch` sequences on H / BR workgroups per set: as many sets as the compute units hold (at most one per sequence),
// then several sequences per workgroup
inline void seq_split(int64_t H, int BR, int batch, int cus, int *sets, int *per_wg) {
    const int64_t wgs = H / BR;
    int g = (int)std::min<int64_t>(batch, std::max<int64_t>(1, cus / wgs));
    const int spb = (batch + g - 1) / g;
    *per_wg = spb;
    *sets = (batch + spb - 1) / spb;
}

// Exchange words of a call: two slots of one word per hidden unit and pair of a workgroup's sequences, for every set
inline int64_t seq_call_words(int64_t H, int sets, int per_wg) { return (int64_t)sets * 2 * ((per_wg + 1) / 2) * H; }
// Words, a claim's among them, that a matrix of M rows has for the largest batch of any sequence that it may be part of: one of 4 H rows
// is an LSTM's, one of 3 H rows a GRU's, and 12 n rows can be both in turn.
inline int64_t seq_exchange_words(int64_t M) { return seq_call_words(M / 3, kSeqMaxBatch, 1) + kSeqClaimWords; }

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

// Forms of a call: sets in grid.y, placed as above, or claimed by the XCDs (seq_claim below).  Claimed are sets of workgroups that an
// XCD's 32 compute units hold one each of, in sequences long enough to pay for the claim: a step on one XCD is 0.4 to 0.6 us
// shorter than one across them, the claim takes 3 to 4 us for one set, 4 to 5 for up to eight, up to 8 for 25.  us per call in the plain
// order / claimed, of 8, 10, 12, 16 steps (LSTM, 32-row blocks): 1024 units, one sequence 21.2 / 21.8, 25.2 / 24.9, 29.3 / 28.2, 37.3 / 34.6;
// seven 21.9 / 22.9, 26.1 / 26.1, 30.1 / 29.3, 38.4 / 35.5; 256 units, one 21.4 / 18.7; twelve 21.0 / 22.1, 24.9 / 25.3, 28.8 / 28.3, 36.5 / 33.8;
// 25 of them 21.0 / 24.0, 24.8 / 26.7, 28.7 / 29.5, 36.5 / 34.9.  Of 64 steps, one sequence of 1024 / 512 / 256 units 128 / 125 / 130 -> 110 / 104 / 95.
// What it costs where other work fills the chip: the call ends when its last workgroup has had a compute unit, also those that have nothing
// to do.  Beside products of 4096 x 4096 on another stream one sequence of 1024 units takes 123 / 131 us for 16 steps, 177 / 213 for 64, three
// 115 / 145 and 187 / 240; 256 units (64 workgroups, not 256) 116 / 113 and 167 / 144.
constexpr int kSeqPlain = 0, kSeqPlaced = 1, kSeqClaimed = 2;
GRIM_HOST_DEVICE bool seq_sets_claimed(int sets, int64_t wgs, int steps) {
    return sets % 8 != 0 && wgs > 1 && (sets + 7) / 8 * wgs <= 32 && steps >= (sets > 8 ? 16 : wgs > 16 ? 10 : 8);
}

// How the workgroups of claimed sets come together.  Every XCD gets as many workgroups, enough for all sets between them (up to eight
// times as many as the sets have), and as soon as a set's worth of them runs on an XCD they take a set.  All of them wait until
// every set is taken; those that are in none then leave.  A call that runs alone thus has each set on one XCD, where words stay in
// its L2.  Where calls overlap and no set fills up -- each could hold some of the compute units and wait for the rest -- a
// workgroup that has waited long enough calls it off, and the first workgroups to ask, wherever they run, make up the sets: the
// call then waits for no more workgroups to run at once than in the plain order.
constexpr int kSeqClaimSlots = 31;                                 // sets' worths of one XCD that can take a set: no call has more sets to claim
struct SeqClaim {
    struct Xcd { unsigned int arrived, owns[kSeqClaimSlots]; } xcd[16];   // workgroups that run; the set that each wgs of them have taken, plus one
    unsigned int complete, ready, mode, asked;                     // sets' worths that run; that have a set; kClaim*; workgroups that asked
};
constexpr unsigned int kClaimPlaced = 1, kClaimSpread = 2;         // SeqClaim::mode (0: open)
// Reads of the mode (1 us each) before a workgroup calls it off: less than the shortest claimed sequence takes.  A call that runs alone needs
// no more than eight (four call off one of 1024 units: 110 -> 128 us); 8 to 64 are alike beside other work.  A caller's own limit on
// the reads of a wait shortens this one in proportion.
constexpr int kSeqClaimPolls = 16;
GRIM_HOST_DEVICE int seq_claim_polls(uint32_t max_polls) { return (int)(max_polls >> 15) < kSeqClaimPolls ? (int)(max_polls >> 15) : kSeqClaimPolls; }

// One thread of a workgroup that runs on XCD `xcd`: its set and its number in the set, or set -1: not needed.  The words are reached
// through `memory`, whose operations are single atomic accesses.
template <class Memory>
GRIM_HOST_DEVICE void seq_claim(SeqClaim *c, const Memory &memory, unsigned int xcd, int sets, int wgs, int max_polls, int *set, int *unit) {
    SeqClaim::Xcd *const x = &c->xcd[xcd & 15u];
    const int number = (int)memory.add_one(&x->arrived);
    const int slot = number / wgs;
    if (number % wgs == wgs - 1 && slot < kSeqClaimSlots) {
        const unsigned int k = memory.add_one(&c->complete);
        if ((int)k < sets) {
            // (acknowledged before it is counted, so that whoever sees the mode sees it; read on this XCD only)
            memory.store_and_wait(&x->owns[slot], k + 1);
            if ((int)memory.add_one(&c->ready) == sets - 1) (void)memory.set_if_zero(&c->mode, kClaimPlaced);
        }
    }
    unsigned int mode = 0;
    for (int polls = 0; polls < max_polls && mode == 0; ++polls) {
        if (polls) memory.pause();
        mode = memory.load(&c->mode);
    }
    if (mode == 0) {
        mode = memory.set_if_zero(&c->mode, kClaimSpread);
        if (mode == 0) mode = kClaimSpread;
    }
    if (mode == kClaimPlaced) {
        *set = slot < kSeqClaimSlots ? (int)memory.load(&x->owns[slot]) - 1 : -1;
        *unit = number % wgs;
    } else {
        const int asked = (int)memory.add_one(&c->asked);
        *set = asked < sets * wgs ? asked / wgs : -1;
        *unit = asked % wgs;
    }
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
