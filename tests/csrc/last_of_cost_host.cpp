// csrc/last_of_cost.h for the host: a row of cells as a segment's first layer stores it, entry by entry in the given order.
#include "../../paper_2312_08053_amd/csrc/last_of_cost.h"

extern "C" uint32_t store_row(const uint32_t* costs, const double* errors, uint32_t n, const uint32_t* order, double* row) {
    uint32_t stores = 0;
    for (uint32_t x = 0; x < n; ++x) {
        const uint32_t k = order[x];
        if (!kimad::last_of_cost(k, n, [&](uint32_t i) { return costs[i]; })) continue;
        row[costs[k]] = errors[k];
        ++stores;
    }
    return stores;
}
