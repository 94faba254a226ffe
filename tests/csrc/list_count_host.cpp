// csrc/list_count.h for a host test.
#include "../../paper_2312_08053_amd/csrc/list_count.h"

extern "C" uint64_t count(const uint32_t* ktab, uint64_t L, uint64_t J, uint64_t unit, uint64_t cap, uint64_t limit) {
    return kimad::count_list_records(ktab, L, J, unit, cap, limit);
}
