// Which of a layer's kept list entries stands for its cost, the same on host and device.
#pragma once
#include <cstdint>

namespace kimad {

// Kept entries come with costs that do not fall and errors that do.  Two of them have the same cost where a caller's errors rise inside
// a run of equal costs (5, 3, 7, 1: two runs, and 1 < 3): the later one's error is the least at that cost.  Entries stored side by side,
// a lane each, must be of different costs: true for one entry of each.  cost(k): entry k's, k < n.
template <typename Cost>
constexpr bool last_of_cost(uint32_t k, uint32_t n, Cost cost) {
    return k + 1u >= n || cost(k + 1u) != cost(k);
}

}  // namespace kimad
