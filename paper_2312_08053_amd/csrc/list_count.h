// How many candidate-list records an allocation will have, counted on the host before it is enqueued.
#pragma once
#include <cstdint>

namespace kimad {

// ktab: L rows of J sizes, each row ascending and at least 1.  Counts the different costs ceil(size / unit) up to `cap` of every
// row, and stops above `limit`.
// The budget of a round decides unit and cap, so a caller whose budget changes pays for this in every call: one product a
// size in place of a division (a quotient of 32 bits by `unit` is the upper half of the product with ceil(2^64 / unit),
// exactly for every unit).  148 to 1024 layers with 64 ratios: 35 to 57 us by divisions, 10 to 17 so.
inline uint64_t count_list_records(const uint32_t* ktab, uint64_t L, uint64_t J, uint64_t unit, uint64_t cap, uint64_t limit) {
    const uint64_t inverse = unit > 1u ? ~0ull / unit + 1u : 0u;
    uint64_t records = 0;
    for (uint64_t i = 0; i < L && records <= limit; ++i) {
        uint64_t last = 0;
        for (uint64_t j = 0; j < J; ++j) {
            const uint64_t v = ktab[i * J + j] - 1u;
            const uint64_t w = 1u + (unit > 1u ? (uint64_t)(((unsigned __int128)v * inverse) >> 64) : v);
            if (w > cap) break;
            records += w != last;
            last = w;
        }
    }
    return records;
}

}  // namespace kimad
