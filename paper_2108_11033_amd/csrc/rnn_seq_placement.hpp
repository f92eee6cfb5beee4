// Which sets of workgroups of the sequence kernel are placed on an XCD of their own, and how.
#pragma once
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

}  // namespace grim
