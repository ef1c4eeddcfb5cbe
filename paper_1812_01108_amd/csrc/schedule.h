// Scan schedules as plain values, and the ones the autotuner tries (no device
// types here: the list is tested on the host alone).
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

namespace a2c {

// Residues per lane and waves per workgroup.
struct Shape {
    int32_t K, W;
    bool operator==(const Shape &o) const { return K == o.K && W == o.W; }
};

// The autotuner's candidates in the order they are timed: the plan's default
// schedule and its present one (the default rules take any number of waves,
// which the grid does not), so that tuning never leaves a plan with a schedule
// that timed slower than what it had; then a grid, fewest residues per lane
// first.  The setters' checks drop what a kernel does not take.
inline std::vector<Shape> tune_candidates(Shape def, Shape now)
{
    std::vector<Shape> c{def};
    const auto add = [&](Shape s) {
        if (std::find(c.begin(), c.end(), s) == c.end()) c.push_back(s);
    };
    add(now);
    for (int32_t k : {1, 2, 4, 8})
        for (int32_t w : {1, 2, 3, 4, 6, 8, 12, 16}) add({k, w});
    return c;
}

}  // namespace a2c
