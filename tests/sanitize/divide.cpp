// The division by a number whose inverse was made beforehand (csrc/xcd_map.hpp), on the host.
#include "xcd_map.hpp"

// quotients of n and its neighbours by d that are wrong
extern "C" int divide_faults(int n, int d) {
    const uint32_t inverse = grim::divide_inverse(d);
    int wrong = 0;
    for (int64_t m = (int64_t)n - 2; m <= (int64_t)n + 2; ++m)
        if (m >= 0 && m <= 0x7fffffff && grim::divide_by((int)m, d, inverse) != (int)(m / d)) ++wrong;
    return wrong;
}
