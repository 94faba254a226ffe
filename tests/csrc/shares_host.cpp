// csrc/shares.h for the host, behind a C interface.
#include "../../paper_2312_08053_amd/csrc/shares.h"

extern "C" uint32_t shares(const uint32_t* ends, uint32_t layers, uint32_t wgs, uint32_t* out, uint32_t room) {
    const std::vector<uint32_t> first = kimad::plan_shares(std::vector<uint32_t>(ends, ends + layers), wgs);
    for (size_t i = 0; i < first.size() && i < room; ++i) out[i] = first[i];
    return (uint32_t)first.size();
}
