// Arithmetic of a segment of the streaming pass (a workgroup's share of a layer), the same on host and device: how far it may
// go with one histogram, and how the space for its candidates is handed out.
//
// Histogram.  A packed histogram entry counts to 2^20 - 1, which any PK_MAX_CHUNKS chunks fit.  Real layers spread over thousands of
// entries: before a stretch ends, one wave reads the counts and allows as many more chunks as the fullest entry has room
// for, whatever they hold, while the others go on.  Only where that is next to nothing does the stretch end there, with a
// part written out and the histogram cleared.
// (Parts at every 1023 chunks were 212 MB for 10 GB of g and h, and every one of them emptied the compute unit.)
#pragma once
#include <cstdint>

namespace kimad {

constexpr uint32_t CHUNK = 1024;              // elements one wave compacts at a time (4 quads per lane)
constexpr uint32_t PK_MAX_COUNT = 0xFFFFF;    // largest count of a packed histogram entry
constexpr uint32_t PK_MAX_CHUNKS = PK_MAX_COUNT / CHUNK;     // (1023)

enum : uint32_t { LIMIT_FREE = 0, LIMIT_READING = 1, LIMIT_FINAL = 2 };
constexpr uint32_t LIMIT_NEAR = 64;             // chunks before the limit at which a wave sees to it
constexpr uint32_t LIMIT_LEAST = 128;           // chunks that are worth going on for

// Whether a stretch that may count the chunks below `allowed` goes on, and up to where.  `most`: the fullest entry's count,
// read after `taken`, the first chunk that nobody had taken; of the chunks before it up to `open` may be missing from the
// count.  Those count against the room like the ones to come: without room for them the limit stays, also where the
// segment has no further chunks (`taken` passes its end while up to `open` of them are still to be counted).
struct StretchLimit { uint32_t end; bool on; };
constexpr StretchLimit stretch_limit_after(uint32_t seg_end, uint32_t allowed, uint32_t taken, uint32_t most, uint32_t open) {
    const uint32_t room = (PK_MAX_COUNT - most) / CHUNK;
    if (room <= open) return {allowed, false};
    const uint32_t reach = taken + (room - open), end = reach < seg_end ? reach : seg_end;
    return {end, end == seg_end || end >= allowed + LIMIT_LEAST};
}

// The limit below which a wave that holds `chunk` may count, as far as it has to know it: final, or well beyond the chunk.
// W, a wave's view of what the workgroup shares: state(), allowed(), taken(), most(), claim() (LIMIT_FREE -> LIMIT_READING,
// by one wave), allow(end), release(state), pause().
// The limit is read again before anything is done about it: the waves that come near the same limit find it lifted by the
// first of them, and one that claims the reading all the same finds out and lets go.  (Without that the second one met a
// limit that was as far as the counts went already and ended the stretch, at about 1950 chunks whatever they hold: 869
// parts on the Llama-shaped set for the 424 of one per workgroup and layer; step 2815 -> 2795 us.)
template <typename W>
constexpr uint32_t stretch_limit(W& w, uint32_t chunk, uint32_t limit, uint32_t seg_end, uint32_t open) {
    while (limit < seg_end && chunk + LIMIT_NEAR >= limit) {
        const uint32_t state = w.state();
        limit = w.allowed();                              // (read after the state: final with it)
        if (state == LIMIT_FINAL || limit == seg_end || chunk + LIMIT_NEAR < limit) break;
        if (state == LIMIT_READING) {
            if (chunk < limit) break;                     // another wave sees to it
            w.pause();
        } else if (w.claim()) {
            uint32_t next = LIMIT_FREE;
            if (w.allowed() == limit) {
                const uint32_t taken = w.taken();         // (before the counts are read)
                const StretchLimit l = stretch_limit_after(seg_end, limit, taken, w.most(), open);
                if (l.on) w.allow(l.end);
                else next = LIMIT_FINAL;
            }
            w.release(next);
        }
    }
    return limit;
}

// ---- candidates ----------------------------------------------------------------------------------
// The segment owns REGION_PER_CHUNK entries of the layer's region per chunk, a third more than the eighth of a layer that
// k_predict lets spill.  A wave takes a block of `block` entries for the chunks of up to SPILL_RUN candidates, and for a
// denser chunk as many units as hold it.
// Units are 128-byte lines of values, from the first whole one of the slice on; but of a slice of a few chunks lines would
// take what the third is there for: a chunk of 129 candidates takes 160 entries and a slice of one chunk may have 128 in
// whole lines, so an eighth of a layer spilled overflowed such slices in up to 23 % of cases, each of which sends the whole
// layer to the passes that read g and h again.  There a unit is eight entries, from the slice's first one: any sixteen
// chunks of up to 168 candidates fit.
// (The blocks that sixteen waves leave nearly empty are 2048 entries below 256 chunks, and at most a tenth of the slice from
// there on.)
constexpr uint32_t REGION_PER_CHUNK = 168;
constexpr uint32_t SPILL_LINE_LOG = 5, SPILL_SHORT_LOG = 3;     // (4-byte values)
constexpr uint32_t SPILL_SHORT = 128;           // chunks below which a slice is handed out in short units
constexpr uint32_t SPILL_RUN = 64;              // candidates a wave writes at a time

struct SpillSlice {
    uint32_t first;       // the slice's first entry, relative to the layer's region
    uint32_t unit_log;    // log2 of the entries of a unit
    uint32_t units;
    uint32_t block;
};
// region: first entry of the layer's region (the buffer's start is a line's)
constexpr SpillSlice spill_slice(uint64_t region, uint32_t first_chunk, uint32_t chunks) {
    const uint32_t first = first_chunk * REGION_PER_CHUNK, log = chunks < SPILL_SHORT ? SPILL_SHORT_LOG : SPILL_LINE_LOG;
    const uint32_t line = 1u << SPILL_LINE_LOG, off = chunks < SPILL_SHORT ? 0u : (line - (uint32_t)((region + first) % line)) % line;
    return {first + off, log, (chunks * REGION_PER_CHUNK - off) >> log, chunks >= 512u ? 512u : chunks >= 256u ? 256u : 128u};
}

}  // namespace kimad
