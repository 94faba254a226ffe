// The streaming pass in shares of chunks, one a workgroup: consecutive chunks of consecutive layers.
//
// A share costs its chunks and SHARE_SEGMENT for every layer that it has a part of: the layer's record, an empty histogram, the first
// loads, the last wave's chunk, the part's stores, 6 to 9 us where a chunk of a full chip takes 0.3.  The kernel ends with its
// dearest share, so that one is made as cheap as can be, but for SHARE_LEAST chunks of a layer: a part is written out whole.
// (Shares of equal numbers of chunks: of ResNet-50's 97 chunks a workgroup 215 lay in one layer and ended after 41 us, one in
// five layers, after 71.  Steps, us, with equal shares and SHARE_SEGMENT 8, 16, 24, 32, 48: ResNet-50 222, 200, 195, 196, 197, 197,
// with a wide link 288, 267, 260, 259, 260, 260, ResNet-18 with 50 ratios 230, 209, 204, 206, 206, 206, with 5 274, 258, 257,
// 257, 257, 257; GPT-2-shaped, 475 chunks a workgroup, 384 to 389 whatever it is.  A perceptron of 266 K elements, with equal shares and
// SHARE_LEAST 8, 16, 32: 108, 98, 98, 102.)
#pragma once
#include <algorithm>
#include <cstdint>
#include <vector>

namespace kimad {

constexpr uint32_t SHARE_SEGMENT = 20, SHARE_LEAST = 16;

// Cuts the layers (`ends`: the chunk behind each one's last) into shares of at most `cost`, each as long as that allows: no other
// cut takes fewer.  Returns their number; first (not null): the chunk where each begins.
inline uint32_t cut_shares(const std::vector<uint32_t>& ends, uint64_t cost, std::vector<uint32_t>* first) {
    uint32_t count = 0, cur = 0;
    for (size_t b = 0; b < ends.size(); ++count) {
        if (first) first->push_back(cur);
        for (uint64_t left = cost; b < ends.size() && left > SHARE_SEGMENT;) {
            const uint32_t taken = (uint32_t)std::min<uint64_t>(left - SHARE_SEGMENT, ends[b] - cur);
            left -= SHARE_SEGMENT + taken;
            cur += taken;
            if (cur == ends[b]) ++b;
        }
    }
    return count;
}

// The chunks where the shares of at most `wgs` workgroups begin.
inline std::vector<uint32_t> plan_shares(const std::vector<uint32_t>& ends, uint32_t wgs) {
    uint64_t lo = SHARE_SEGMENT + SHARE_LEAST;
    uint64_t hi = ends.empty() ? lo : std::max<uint64_t>(lo, (uint64_t)SHARE_SEGMENT * ends.size() + ends.back());     // (all in one)
    while (lo < hi) {
        const uint64_t mid = lo + (hi - lo) / 2u;
        if (cut_shares(ends, mid, nullptr) <= wgs) hi = mid; else lo = mid + 1u;
    }
    std::vector<uint32_t> first;
    cut_shares(ends, lo, &first);
    return first;
}

}  // namespace kimad
