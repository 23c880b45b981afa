// The segment cost that the two solvers of the 1-D k-means evaluate.
#pragma once

#include "lanes.h"

namespace gpic {
namespace {

// cost(j, i) from the prefix sums at j and i + 1
__device__ __forceinline__ double seg_cost(double2 a, double2 e, int64_t j, int64_t i)
{
    const double m = (double)(i - j + 1);
    const double s1 = e.x - a.x;
    const double s2 = e.y - a.y;
    const double c = s2 - s1 * s1 / m;
    return c > 0.0 ? c : 0.0;
}

} // namespace
} // namespace gpic
