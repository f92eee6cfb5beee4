// How the workgroups of a launch are dealt to the XCDs.
#pragma once
#include <cstdint>

#include "host_device.hpp"

namespace grim {

// n / d for 0 <= n < 2^31 with `inverse` = divide_inverse(d), made on the host: a launch's numbers are uniform, and a division by
// a run-time value takes the scalar unit thirty instructions and a trip to the vector ALU and back.  The product is short of
// the quotient by one at most: the inverse is short of 2^32 / d by less than two, n below 2^31.
inline uint32_t divide_inverse(int32_t d) { return 0xffffffffu / (uint32_t)(d > 0 ? d : 1); }
GRIM_HOST_DEVICE int divide_by(int n, int d, uint32_t inverse) {
    const int q = (int)(((uint64_t)(uint32_t)n * inverse) >> 32);
    return q + (n - q * d >= d ? 1 : 0);
}

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
    uint32_t per_tile_inv, per_part_inv;
};
inline XcdMap xcd_map(int32_t ntiles, int64_t per_tile, int64_t *nwg) {
    XcdMap m;
    const int32_t full = ntiles / 8, r = ntiles % 8;
    m.per_tile = (int32_t)per_tile;
    m.tail_slot0 = (int32_t)(full * per_tile);
    m.tail_tile0 = full * 8;
    m.shift = r == 0 ? 0 : r % 4 == 0 ? 1 : r % 2 == 0 ? 2 : 3;
    m.per_part = (int32_t)((per_tile + (1 << m.shift) - 1) >> m.shift);
    m.per_tile_inv = divide_inverse(m.per_tile);
    m.per_part_inv = divide_inverse(m.per_part);
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
        const int q = divide_by(slot, m.per_tile, m.per_tile_inv);
        *tile = q * 8 + xcd;
        *unit = slot - q * m.per_tile;
        return true;
    }
    const int s2 = slot - m.tail_slot0;
    const int q = divide_by(s2, m.per_part, m.per_part_inv);
    const int part = q * 8 + xcd;
    *tile = m.tail_tile0 + (part >> m.shift);
    *unit = ((s2 - q * m.per_part) << m.shift) + (part & ((1 << m.shift) - 1));
    return *tile < ntiles;
}

}  // namespace grim
