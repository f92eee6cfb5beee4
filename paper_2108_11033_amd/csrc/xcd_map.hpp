// How the workgroups of a launch are dealt to the XCDs.
#pragma once
#include <cstdint>

#include "host_device.hpp"

namespace grim {

// Workgroup id -> (tile of columns, unit of the tile's work) for the kernels whose workgroups of one
// tile fetch the same rows: ids are dealt to the 8 XCDs round-robin, each XCD has its own L2, so a
// tile's units go to one XCD.  With that alone the last ntiles % 8 tiles (all of them when there
// are fewer than 8: one tile for N <= 64) would leave XCDs idle, so each of those tiles is cut into
// 2^shift interleaved parts, enough for a multiple of 8, and the parts are dealt instead.
struct XcdMap {
    int32_t per_tile;         // units per tile
    int32_t tail_slot0;       // first slot (id / 8) of the tail tiles
    int32_t tail_tile0;       // first tail tile, a multiple of 8
    int32_t shift;            // tail tiles are cut into 1 << shift parts ...
    int32_t per_part;         // ... of this many units
};
inline XcdMap xcd_map(int32_t ntiles, int64_t per_tile, int64_t *nwg) {
    XcdMap m;
    const int32_t full = ntiles / 8, r = ntiles % 8;
    m.per_tile = (int32_t)per_tile;
    m.tail_slot0 = (int32_t)(full * per_tile);
    m.tail_tile0 = full * 8;
    m.shift = r == 0 ? 0 : r % 4 == 0 ? 1 : r % 2 == 0 ? 2 : 3;
    m.per_part = (int32_t)((per_tile + (1 << m.shift) - 1) >> m.shift);
    *nwg = 8 * (full * per_tile + (int64_t)((r << m.shift) / 8) * m.per_part);
    return m;
}

// The same for a launch of many matrices of one tile each (grid.x workgroups to a matrix, grid.y matrices): a workgroup's unit is its
// id, and no id is added, so that ids running on over the matrices are dealt to the XCDs evenly.  With grid.x filled up to a
// multiple of 8 each matrix would begin on the first XCD again, and matrices of two units would run on two XCDs (236 of 32 x 1824 of
// mixed rates at 6 columns 10.1 us, 4.3 this way; 225 of 32 x 3936 at one 12.9, 5.0; 211 of 64 x 1440 keeping 10 x 10 at 5 9.1, 6.2).
inline XcdMap xcd_map_one_tile(int64_t units, int64_t *nwg) {
    const XcdMap m = xcd_map(1, units, nwg);
    *nwg = units;
    return m;
}

// false: the workgroup has no tile
GRIM_HOST_DEVICE bool xcd_map_at(const XcdMap &m, int id, int ntiles, int *tile, int *unit) {
    const int xcd = id & 7, slot = id >> 3;
    if (slot < m.tail_slot0) {
        *tile = (slot / m.per_tile) * 8 + xcd;
        *unit = slot % m.per_tile;
        return true;
    }
    const int s2 = slot - m.tail_slot0;
    const int part = (s2 / m.per_part) * 8 + xcd;
    *tile = m.tail_tile0 + (part >> m.shift);
    *unit = ((s2 % m.per_part) << m.shift) + (part & ((1 << m.shift) - 1));
    return *tile < ntiles;
}

}  // namespace grim
