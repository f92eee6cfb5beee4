// How the workgroups of a launch are dealt to the XCDs (the device's half, xcd_map_at, is in spmm_common.hpp).
#pragma once
#include <cstdint>

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

}  // namespace grim
