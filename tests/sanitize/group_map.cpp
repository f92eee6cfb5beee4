// Groups of matrices on the matrix cores, on the host: a walk over the workgroups of a launch (csrc/xcd_map.hpp) and the rule that sends
// uniformly pruned ones there (csrc/group_rules.hpp).
#include <algorithm>
#include <vector>

#include "group_rules.hpp"
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

// (every run keeps `kept` columns of a column block)
extern "C" int group_on_matrix_cores(int count, int M, int K, int BR, int BC, int kr, int kc, int kept, int batch) {
    const int64_t runs = (M + 15) / 16, steps = (K / BC * kept + 31) / 32;
    return grim::group_quicker_on_matrix_cores(count, M / BR, K / BC, kr, kc, K, runs, count * runs * steps, batch);
}
