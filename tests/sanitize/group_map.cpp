// Host walk over the workgroups of a launch of many matrices of one tile each (csrc/xcd_map.hpp).
#include <algorithm>
#include <vector>

#include "xcd_map.hpp"

// -1: a unit of a matrix is not run by exactly one workgroup; else how many workgroups with work the most loaded XCD has above its
// even share, linear ids being dealt to the eight XCDs in turn
extern "C" int group_map_excess(int units, int count) {
    int64_t nwg = 0;
    const grim::XcdMap m = grim::xcd_map_one_tile(units, &nwg);
    std::vector<int> met((std::size_t)units * count, 0), load(8, 0);
    for (int matrix = 0; matrix < count; ++matrix)
        for (int id = 0; id < nwg; ++id) {
            int tile = -1, unit = -1;
            if (!grim::xcd_map_at(m, id, 1, &tile, &unit) || unit >= units) continue;
            if (tile != 0 || unit < 0) return -1;
            ++met[(std::size_t)matrix * units + unit];
            ++load[(matrix * nwg + id) % 8];
        }
    for (int n : met)
        if (n != 1) return -1;
    return *std::max_element(load.begin(), load.end()) - (units * count + 7) / 8;
}
