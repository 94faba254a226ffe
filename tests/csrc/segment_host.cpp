// The streaming pass's segment arithmetic (csrc/segment.h) for a host test.
#include <atomic>
#include <thread>
#include <vector>

#include "../../paper_2312_08053_amd/csrc/segment.h"

using namespace kimad;

extern "C" {

// out: [0] the new limit, [1] whether the stretch goes on
void limit_after(uint32_t seg_end, uint32_t allowed, uint32_t taken, uint32_t most, uint32_t open, uint32_t* out) {
    const StretchLimit l = stretch_limit_after(seg_end, allowed, taken, most, open);
    out[0] = l.end; out[1] = l.on;
}

// One segment by `waves` threads that walk it as the waves of k_main do: a chunk in hand, one taken ahead, counts added in
// between.  Every chunk has `per[e]` entries of histogram entry e (1024 in all).  out: [0] stretches, [1] largest count of any
// entry at the end of a stretch, [2] chunks counted, [3] stretches that ended apart (the waves disagreed).
void walk(uint32_t waves, uint32_t seg_end, const uint32_t* per, uint32_t entries, uint32_t spin, uint32_t* out) {
    std::vector<std::atomic<uint32_t>> counts(entries);
    std::atomic<uint32_t> next, allowed, state;
    struct View {
        std::vector<std::atomic<uint32_t>>& counts;
        std::atomic<uint32_t>&next_, &allowed_, &state_;
        uint32_t state() const { return state_; }
        uint32_t allowed() const { return allowed_; }
        uint32_t taken() const { return next_; }
        uint32_t most() const {
            uint32_t m = 0;
            for (auto& c : counts) m = c > m ? c.load() : m;
            return m;
        }
        bool claim() const { uint32_t free = LIMIT_FREE; return state_.compare_exchange_strong(free, LIMIT_READING); }
        void allow(uint32_t end) const { allowed_ = end; }
        void release(uint32_t s) const { state_ = s; }
        void pause() const { std::this_thread::yield(); }
    };
    out[0] = out[1] = out[2] = out[3] = 0;
    for (uint32_t start = 0; start < seg_end;) {
        for (auto& c : counts) c = 0;
        next = start + waves;
        allowed = seg_end < start + PK_MAX_CHUNKS ? seg_end : start + PK_MAX_CHUNKS;
        state = LIMIT_FREE;
        std::vector<uint32_t> stop(waves);
        std::atomic<uint32_t> done{0};
        std::vector<std::thread> threads;
        for (uint32_t k = 0; k < waves; ++k)
            threads.emplace_back([&, k] {
                View v{counts, next, allowed, state};
                uint32_t chunk = start + k, limit = allowed;
                for (uint32_t n = 0;; ++n) {
                    if (limit < seg_end && chunk + LIMIT_NEAR >= limit) limit = stretch_limit(v, chunk, limit, seg_end, 2u * waves);
                    if (chunk >= limit) break;
                    const uint32_t taken = next++;
                    for (volatile uint32_t s = 0; s < spin * ((k * 7u + n * 13u) % 17u); s = s + 1) {}   // (uneven paces)
                    for (uint32_t e = 0; e < entries; ++e) counts[e] += per[e];
                    ++done;
                    chunk = taken;
                }
                stop[k] = limit;
            });
        for (auto& t : threads) t.join();
        for (uint32_t k = 1; k < waves; ++k) out[3] += stop[k] != stop[0];
        for (auto& c : counts) out[1] = c > out[1] ? c.load() : out[1];
        out[0] += 1;
        out[2] += done;
        start = stop[0];
    }
}

// A slice's chunks, of counts[k] candidates each, taken in turn by the wave order[k] says, as main_chunk takes space for them.
// out: [0] first entry, [1] one past the last entry handed out, [2] whether all of them fitted.
void spill(uint64_t region, uint32_t first_chunk, uint32_t chunks, const uint32_t* counts, const uint32_t* order, uint32_t* out) {
    const SpillSlice s = spill_slice(region, first_chunk, chunks);
    uint32_t cursor = 0, fill[16], last = s.first;
    bool have[16] = {}, fits = true;
    auto take = [&](uint32_t entries) {
        const uint32_t b = cursor, n = (entries + (1u << s.unit_log) - 1u) >> s.unit_log;
        cursor += n;
        const bool ok = b + n <= s.units;
        if (ok) last = s.first + ((b + n) << s.unit_log);
        return ok;
    };
    for (uint32_t k = 0; k < chunks; ++k) {
        const uint32_t n = counts[k], w = order[k];
        if (n > SPILL_RUN) {
            fits = take(n) && fits;
        } else if (n) {
            if (!have[w] || fill[w] + n > s.block) { have[w] = take(s.block); fill[w] = 0; fits = have[w] && fits; }
            fill[w] += n;
        }
    }
    out[0] = s.first; out[1] = last; out[2] = fits;
}

}  // extern "C"
