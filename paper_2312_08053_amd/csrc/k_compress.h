// Selection, compaction and estimator update.
//
// Computes, per layer, the support of TopK_K(x) for x = g - h (paper Section 2.2), writes the
// (index, value) payload that Algorithm 1's worker uploads, and applies h <- h + TopK(x)
// (Section 3.3, Eq. EF21-2).  Equal magnitudes are kept in order of lower index.
//
// Tiled layers: one streaming pass writes every entry whose 19-bit key prefix is >= the layer's
// threshold prefix into a candidate buffer (in index order inside each 1024-element chunk) and
// histograms the last 12 key bits of the entries whose prefix is equal.  Four small kernels then
// fix the exact threshold key and tie quota, count survivors per chunk, scan the chunks in index
// order and write payload and estimator.
#pragma once
#include "common.h"
#include <hip/hip_fp16.h>
#include "k_profile.h"

namespace kimad {

struct CompressBuffers {
    const LayerDesc* layers;
    const uint32_t* chunk_layer;  // tile -> layer (a tile holds tile_elems / CHUNK chunks)
    const uint32_t* big_layer;
    const uint32_t* small_layer;
    uint32_t tile_elems;
    uint32_t L, B, J;
    const uint32_t* Ktab;         // [L][J] grid sizes
    // threshold cache written by the profile scans
    const uint32_t* sel_prefix;
    const uint32_t* sel_above;
    const uint32_t* sel_amb;
    // per big layer
    SelRec* sel;                  // [B]
    uint32_t* cursor;             // [B] candidates reserved so far
    uint32_t* hist3;              // [B][4096] last-digit histogram of the ambiguous entries
    uint32_t* tau;                // [B] exact threshold key
    uint32_t* quota;              // [B] entries equal to tau that are kept (lowest indices)
    // per chunk
    uint32_t* rec_start;          // start inside the layer's candidate region
    uint32_t* rec_cnt;            // candidates written
    uint32_t* rec_amb;            // of which ambiguous
    uint32_t* c_gt;               // candidates above tau
    uint32_t* c_eq;               // candidates equal to tau
    uint32_t* o_base;             // first payload slot of the chunk inside the layer
    uint32_t* o_allow;            // ties this chunk may keep
    const uint32_t* chunk_first;  // chunk -> first chunk of its layer (with the big index: where its region starts)
    const uint32_t* cblk_big;     // block of 1024 chunks -> big index
    // candidate buffer: x, and its position in the chunk's 1024
    float* tmp_x;
    uint16_t* tmp_i;
    uint32_t* ncompact;       // [0] layers whose selection needs the streaming compaction pass, [1] of which served from g and h throughout (SEL_DIRECT)
    uint32_t* fresh;          // 1 while the profile's cache describes the current g - h (see ProfileBuffers)
    const LayerState* state;      // fused-profile state (spill range) per big layer
    // outputs
    const uint64_t* K;
    const uint64_t* offsets;
    uint32_t* idx_out;
    float* val_out;               // fp32 values, or binary16 bit patterns (uint16) when value_f16 is set
    uint32_t value_f16;
    uint64_t capacity_pairs;
    uint64_t tmp_total;           // entries of the candidate buffer (all regions)
    int32_t* status;
};

// A kept value as it travels in half precision: binary16, round to nearest even, saturated to +-65504 (never
// infinite), NaN kept.  Returns the bit pattern; *decoded gets the fp32 value the receiver will add.
__device__ __forceinline__ uint16_t value_to_f16(float x, float* decoded) {
    const float c = x != x ? x : fminf(fmaxf(x, -65504.f), 65504.f);
    const __half hv = __float2half_rn(c);
    *decoded = __half2float(hv);
    return __half_as_ushort(hv);
}

// Payload slot o gets value x; returns what the estimator must add: x itself, or its half-precision image.
__device__ __forceinline__ float emit_value(const CompressBuffers& cb, uint64_t o, float x) {
    if (cb.value_f16) {
        float dec;
        reinterpret_cast<uint16_t*>(cb.val_out)[o] = value_to_f16(x, &dec);
        return dec;
    }
    cb.val_out[o] = x;
    return x;
}

// ---------------------------------------------------------------------------------------------
// Per layer: turn K[i] into a selection record using the profile's threshold cache.
// One workgroup, of whose threads the first `threads` are there; thread b handles big layer b (looping).  `reuse`: the
// thresholds are those of an earlier profile; `use_candidates`: a single pass over g and h (that profile's, or this call's own)
// has left candidates.  In kimad_step the allocation's last kernel does this with the sizes that it has just written (after a
// barrier that waits for them), and hands over which grid sizes they are, which a launch of its own has to search for.
// (Walk and look-up, us: two launches 15.0 on the GPT-2-shaped set and 14.9 on ResNet-50, one 13.0 and 13.2; Llama-shaped 20
// and 17.)
// `j` (not null): the grid size that every layer's K is.
__device__ __forceinline__ void lookup(const CompressBuffers& cb, uint32_t threads, int32_t err_offgrid, int32_t err_offsets, int32_t err_stale,
                                       uint32_t reuse, uint32_t use_candidates, const int32_t* j) {
    __shared__ int bad;
    __shared__ uint32_t need_pass, n_direct;
    const uint32_t tid = threadIdx.x;
    // Thresholds may be reused only if a profile wrote them for the g - h that is there now: the compression
    // itself changes h, so a second call without a new profile in between is refused (status err_stale).
    const bool stale = reuse && *cb.fresh != 1u;
    const uint32_t my_layer = tid < cb.B ? cb.big_layer[tid] : 0u;           // (asked for ahead of the barriers)
    if (tid == 0) { bad = stale ? 3 : 0; need_pass = 0u; n_direct = 0u; }
    __syncthreads();
    // validate offsets / K for every layer
    for (uint32_t i = tid; i < cb.L; i += threads) {
        const uint64_t K = cb.K[i], off = cb.offsets[i];
        if (K > cb.layers[i].n || off > cb.capacity_pairs || K > cb.capacity_pairs - off) atomicMax(&bad, 1);
    }
    __syncthreads();
    const bool offsets_bad = bad == 1;
    __syncthreads();
    for (uint32_t b = tid; b < cb.B; b += threads) {
        SelRec r;
        r.mode = SEL_NONE; r.prefix = 0; r.above = 0; r.amb = 0; r.cap = 0; r.K = 0;
        const uint32_t li = b == tid ? my_layer : cb.big_layer[b];
        const LayerDesc ld = cb.layers[li];
        const LayerState st = cb.state[b];
        const uint32_t n = ld.n;
        r.tmp_base = ld.tmp0;
        r.h = ld.h;
        r.mis = ld.mis;
        r.dst = cb.offsets[li];
        if (!offsets_bad && !stale) {
            const uint32_t K = (uint32_t)cb.K[li];
            r.K = K;
            if (K == 0u) {
                r.mode = SEL_NONE;
            } else if (K == n) {
                r.mode = SEL_DIRECT; r.above = n;        // everything is kept: no candidates, no threshold
            } else {
                // the row of grid sizes is read eight entries at a time (a look-up that stops at the
                // first hit would wait for one load per entry)
                int found = -1;
                if (j) {
                    const uint32_t t = min((uint32_t)j[li], cb.J - 1u);
                    if (cb.Ktab[(size_t)li * cb.J + t] == K) found = (int)t;
                }
                for (uint32_t j0 = 0; j0 < cb.J && found < 0; j0 += 8) {
                    uint32_t kt[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) kt[u] = cb.Ktab[(size_t)li * cb.J + min(j0 + (uint32_t)u, cb.J - 1u)];
#pragma unroll
                    for (int u = 7; u >= 0; --u)
                        if (j0 + (uint32_t)u < cb.J && kt[u] == K) found = (int)(j0 + (uint32_t)u);
                }
                if (found < 0) {
                    atomicMax(&bad, 2);
                } else {
                    const size_t t = (size_t)li * cb.J + found;
                    r.prefix = cb.sel_prefix[t];
                    r.above = cb.sel_above[t];
                    r.amb = cb.sel_amb[t];
                    r.cap = ld.tmp_cap;
                    // every entry at or above the threshold prefix already sits in the candidate buffer
                    const bool in_spill = use_candidates && st.spill_valid && st.spill_bin < D1_BINS &&
                                          r.prefix >= (st.spill_bin << D2_BITS);
                    // The compaction pass writes what lies at or above the threshold prefix into the region; its
                    // waves reserve space in blocks and leave a block's tail unused when the next chunk does not
                    // fit (less than the chunk needs, so at most as much again), and every wave its last block
                    // of a tile.  What would not fit is served from g and h directly.
                    const uint64_t need = 2ull * ((uint64_t)r.above + r.amb) + 4ull * SPILL_BLOCK * ld.ntiles;
                    r.mode = in_spill ? SEL_CAND : need <= r.cap ? SEL_PREFIX : SEL_DIRECT;
                }
            }
        }
        cb.sel[b] = r;
        // the classic pass reserves its candidates from zero; the spilled ones keep their records
        if (r.mode != SEL_CAND) cb.cursor[b] = 0u;
        if (r.mode == SEL_PREFIX || r.mode == SEL_DIRECT) atomicAdd(&need_pass, 1u);
        if (r.mode == SEL_DIRECT) atomicAdd(&n_direct, 1u);
    }
    __syncthreads();
    if (tid == 0) { cb.ncompact[0] = bad ? 0u : need_pass; cb.ncompact[1] = bad ? 0u : n_direct; }
    if (bad) {
        // refuse the whole call: nothing is written by the later kernels
        for (uint32_t b = tid; b < cb.B; b += threads) { cb.sel[b].mode = SEL_NONE; cb.sel[b].cap = 0; cb.sel[b].K = 0; }
        if (tid == 0) *cb.status = stale ? err_stale : offsets_bad ? err_offsets : err_offgrid;
    } else if (tid == 0) {
        *cb.status = 0;
    }
    // From here on the cache no longer describes g - h (the estimator is about to change, or a selection from
    // scratch has overwritten the cache); a refused call that reuses the profile leaves both as they were.
    if (tid == 0 && (!reuse || !bad)) *cb.fresh = 0u;
}

__global__ __launch_bounds__(256) void k_lookup(CompressBuffers cb, int32_t err_offgrid, int32_t err_offsets,
                                                int32_t err_stale, uint32_t reuse, uint32_t use_candidates) {
    lookup(cb, 256u, err_offgrid, err_offsets, err_stale, reuse, use_candidates, nullptr);
}

// What the allocation's last kernel looks up in kimad_step (on: 0 elsewhere).
struct StepLookup {
    CompressBuffers cb;
    const int32_t* j;
    int32_t err_offgrid, err_offsets, err_stale;
    uint32_t on;
};
__device__ __forceinline__ void step_lookup(const StepLookup& sl, uint32_t threads) {
    if (!sl.on) return;
    __syncthreads();                                     // the sizes and offsets are there
    lookup(sl.cb, threads, sl.err_offgrid, sl.err_offsets, sl.err_stale, 1u, 1u, sl.j);
}

// A value that is the same in every lane, in scalar registers.
template <typename T>
__device__ __forceinline__ T uniform(const T& v) {
    static_assert(sizeof(T) % 4 == 0, "whole registers");
    uint32_t w[sizeof(T) / 4];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (size_t k = 0; k < sizeof(T) / 4; ++k) w[k] = (uint32_t)__builtin_amdgcn_readfirstlane((int)w[k]);
    T r;
    __builtin_memcpy(&r, w, sizeof(T));
    return r;
}

// ---------------------------------------------------------------------------------------------
// Streaming compaction pass (layers whose threshold lies below the spilled range, or all layers
// when no fused profile preceded).  One wave per chunk; a workgroup of 4 waves walks the chunks
// of one tile.  Each lane holds 4 quads (16 elements); positions come from ballots, so
// the candidates of a chunk are written in index order at a range reserved with one atomic.
// Tiles are taken in a grid-stride loop; *cb.ncompact (set by k_lookup) is the number of layers that
// need this pass, so that after a single-pass profile, when the candidates serve every layer, a
// small grid leaves after one load.
// A threshold among zeros or equal values makes nearly every entry ambiguous, with one last digit: sixteen atomics per
// chunk on one word then set the time, 12 ns each, not the read of g and h.  A wave counts such a run in a register and
// a workgroup adds it once: 425 -> 22 us for a layer of 2.4 M entries that are zero but for a 67th, 6.85 ms -> 65 us for
// 38.6 M.
// The layer's records are in scalar registers, x alone is kept of g and h, and a mask holds a lane's sixteen verdicts: 96
// registers for five waves a SIMD, where records in vector registers and Quads took 118 for four, which the candidates'
// half of the launch had to live with too (38.6 M entries without ties 78 -> 58 us; 1.3 billion entries served from
// candidates 57 -> 50).  Six and eight waves cost scratch memory here: 111 and 181 us.
// (Workgroups `block` of `nblocks` of the launch that also histograms the spilled candidates: k_candidates.)
__device__ __forceinline__ void compact_tiles(const CompressBuffers& cb, uint32_t ntiles, int32_t err_internal,
                                              uint32_t block, uint32_t nblocks) {
    if (*cb.ncompact == 0u) return;
    const uint32_t wave = uniform(threadIdx.x >> 6), lane = lane_id();
    const uint32_t chunks_per_tile = cb.tile_elems / CHUNK;
    __shared__ uint32_t* tie_at[4];
    __shared__ uint32_t tie_n[4];
    uint32_t* held_at = nullptr;                // (the same in all lanes)
    uint32_t held_n = 0u;
    for (uint32_t tile = block; tile < ntiles; tile += nblocks) {
    // (the same in every lane, and said so: in vector registers they left the launch four waves a SIMD)
    const uint32_t li = uniform(cb.chunk_layer[tile]);
    const LayerDesc L = uniform(cb.layers[li]);
    const SelRec S = uniform(cb.sel[L.big]);
    const uint32_t tile_in_layer = tile - L.tile0;
    uint32_t* hist3 = cb.hist3 + (size_t)L.big * D3_BINS;
    // layers served from the spilled candidates (or with K = 0) need no pass over g, h
    if (S.mode == SEL_NONE || S.mode == SEL_CAND) continue;
    WaveAlloc wa{0u, 0u};

    for (uint32_t cc = wave; cc < chunks_per_tile; cc += 4) {
        const uint32_t chunk_in_layer = tile_in_layer * chunks_per_tile + cc;
        if (chunk_in_layer >= L.nchunks) break;
        const uint32_t chunk = L.chunk0 + chunk_in_layer;
        const uint32_t vbase = chunk_in_layer * CHUNK;
        if (S.mode == SEL_DIRECT && S.amb == 0u) {
            // everything is kept: the count follows from the layer's ends, nothing is read
            const uint32_t v0 = max(vbase, L.mis), v1 = min(vbase + CHUNK, L.mis + L.n);
            const uint32_t inside = v1 > v0 ? v1 - v0 : 0u;
            if (lane == 0) {
                cb.rec_start[chunk] = 0u; cb.rec_cnt[chunk] = inside; cb.rec_amb[chunk] = 0u;
                cb.c_gt[chunk] = inside; cb.c_eq[chunk] = 0u;
            }
            continue;
        }
        float x[NQ][4];
        // bit 4 u + c: the entry is a candidate; it shares the threshold's prefix
        uint32_t sel = 0, ambig = 0;
        {
            QuadGH q[NQ];
            uint32_t valid;
            load_chunk<(int)NQ>(L, vbase, q, valid);
#pragma unroll
            for (int u = 0; u < (int)NQ; ++u)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    x[u][c] = q[u].g[c] - q[u].h[c];
                    const uint32_t p = key_of(x[u][c]) >> D2_SHIFT, bit = (valid >> (4 * u + c)) & 1u;
                    sel |= (p >= S.prefix ? bit : 0u) << (4 * u + c);
                    ambig |= (p == S.prefix ? bit : 0u) << (4 * u + c);
                }
        }
        // wave totals and the exclusive prefix of the lanes' counts, per quad row
        uint32_t total = 0, total_amb = 0;
        uint32_t rowbase[NQ];                   // candidates in earlier rows + earlier lanes of this row
#pragma unroll
        for (int u = 0; u < (int)NQ; ++u) {
            const uint32_t cnt = __popc((sel >> (4 * u)) & 15u);
            // exclusive prefix over lanes of a small integer: three ballots on its bits
            const uint64_t b0 = ballot(cnt & 1u), b1 = ballot(cnt & 2u), b2 = ballot(cnt & 4u);
            const uint32_t ex = mbcnt(b0) + 2u * mbcnt(b1) + 4u * mbcnt(b2);
            rowbase[u] = total + ex;
            total += __popcll(b0) + 2u * __popcll(b1) + 4u * __popcll(b2);
        }
        {
            uint32_t a = __popc(ambig);
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) a += __shfl_xor(a, d, 64);
            total_amb = a;
        }
        const bool direct = S.mode == SEL_DIRECT;   // counted only: the later kernels read g and h again
        uint32_t start = 0;
        if (total && !direct) start = wave_reserve(wa, total, &cb.cursor[L.big]);
        // k_lookup sends a layer here only if its region holds every chunk's block; should a reservation
        // still not fit, drop it, never write out of bounds, and report it.
        const uint32_t written = direct ? total : start >= S.cap ? 0u : min(total, S.cap - start);
        if (written != total && lane == 0) atomicMin(cb.status, err_internal);
        if (lane == 0) { cb.rec_start[chunk] = start; cb.rec_cnt[chunk] = written; cb.rec_amb[chunk] = total_amb; }
        if (total == 0) continue;
        const uint64_t base = S.tmp_base + start;
        if (!direct) {
#pragma unroll
        for (int u = 0; u < (int)NQ; ++u) {
            uint32_t pos = rowbase[u];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if ((sel >> (4 * u + c)) & 1u) {
                    if ((uint64_t)start + pos < S.cap) {
                        const uint64_t o = base + pos;
                        cb.tmp_x[o] = x[u][c];
                        cb.tmp_i[o] = (uint16_t)(u * 256u + lane * 4u + c);
                    }
                    ++pos;
                }
            }
        }
        }
        if (total_amb) {
#pragma unroll
            for (int u = 0; u < (int)NQ; ++u) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const bool a = (ambig >> (4 * u + c)) & 1u;
                    const uint64_t am = ballot(a);
                    if (am == 0) continue;
                    const uint32_t low = key_of(x[u][c]) & (D3_BINS - 1);
                    // every ambiguous lane holds the same key (zeros, constants): counted in the wave for as long as
                    // the key stays the same
                    const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)low, __ffsll((long long)am) - 1);
                    const bool uniform = ballot(a && low != first) == 0;
                    if (uniform) {
                        if (held_at != hist3 + first) {
                            if (held_n && lane == 0) atomicAdd(held_at, held_n);
                            held_at = hist3 + first;
                            held_n = 0u;
                        }
                        held_n += (uint32_t)__popcll(am);
                    } else if (a) {
                        atomicAdd(&hist3[low], 1u);
                    }
                }
            }
        }
    }
    }
    // what the waves still hold, one atomic for those that hold the same key
    if (lane == 0) { tie_at[wave] = held_at; tie_n[wave] = held_n; }
    // (LDS only: the records' stores need not be waited for)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (threadIdx.x < 4u && tie_n[threadIdx.x]) {
        uint32_t n = 0u;
        bool lowest = true;
        for (uint32_t w = 0; w < 4u; ++w) {
            const bool same = tie_n[w] != 0u && tie_at[w] == tie_at[threadIdx.x];
            n += same ? tie_n[w] : 0u;
            lowest = lowest && !(same && w < threadIdx.x);
        }
        if (lowest) atomicAdd(tie_at[threadIdx.x], n);
    }
}

// ---------------------------------------------------------------------------------------------
// Last-digit histogram of the spilled candidates that share the threshold prefix (layers in
// SEL_CAND mode).  Four lanes per chunk, eight rounds of candidates per memory round trip.
__device__ __forceinline__ void hist3_candidates(const CompressBuffers& cb, uint32_t nchunks_total,
                                                 const uint32_t* chunk_big, uint32_t block) {
    constexpr uint32_t S = SUB_HIST;
    const SubGroup g = sub_group<S>();
    const uint32_t chunk = block * (256u / S) + threadIdx.x / S;
    uint32_t cnt = 0, prefix = 0;
    uint64_t base = 0;
    uint32_t* hist3 = cb.hist3;
    bool is_cand = false;
    if (chunk < nchunks_total) {
        // what the chunk index alone addresses goes out together, then the layer's record
        const uint32_t b = chunk_big[chunk], first = cb.chunk_first[chunk];
        const uint32_t n_rec = cb.rec_cnt[chunk], start = cb.rec_start[chunk];
        materialise(b); materialise(first); materialise(n_rec); materialise(start);
        // where the candidates are follows from the above: they are asked for together with the layer's record
        // (of a layer in another mode in vain: its chunks count as empty)
        base = region_start(first, b) + start;
        // (the compaction half of this launch may be rewriting the records of a layer in another mode: whatever
        // is read of them, nothing is asked for outside the buffer)
        cnt = base + n_rec <= cb.tmp_total ? n_rec : 0u;
        const SelRec S = cb.sel[b];
        is_cand = S.mode == SEL_CAND;
        prefix = S.prefix;
        hist3 = cb.hist3 + (size_t)b * D3_BINS;
    }
    const uint32_t cmax = wave_max_over_groups<S>(cnt);
    uint32_t n_above = 0, n_amb = 0;            // of this chunk: threshold prefix exceeded / shared
    // one round: one candidate of the chunk per lane of its group
    auto round = [&](bool in, uint32_t key) {
        in = in && is_cand;
        const bool a = in && (key >> D2_SHIFT) == prefix;
        const bool hi = in && (key >> D2_SHIFT) > prefix;
        const uint32_t am = ballot_sub<S>(g, a);
        n_above += __popc(ballot_sub<S>(g, hi));
        n_amb += __popc(am);
        if (am == 0) return;
        // one atomic per group when all its matching lanes hold the same key (zeros, constants)
        const uint32_t first = (uint32_t)__ffs((int)am) - 1u;
        const uint32_t k0v = __shfl(key, g.shift + first, 64);
        const bool uniform = ballot_sub<S>(g, a && key != k0v) == 0;
        if (uniform) {
            if (g.sub == first) atomicAdd(&hist3[key & (D3_BINS - 1)], (uint32_t)__popc(am));
        } else if (a) {
            atomicAdd(&hist3[key & (D3_BINS - 1)], 1u);
        }
    };
    // the first eight rounds' loads go out together (positions past the chunk's last candidate read entry 0
    // of the buffer, always a valid address, and are dropped; a chunk without candidates has no valid start)
    // (and so on, eight rounds per memory round trip: a layer that spills an eighth has 32 rounds a chunk)
    constexpr int AHEAD = 8;
    for (uint32_t k0 = 0; k0 < cmax; k0 += AHEAD * S) {
        float px[AHEAD];
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) {
            const uint32_t k = k0 + (uint32_t)t * S + g.sub;
            px[t] = cb.tmp_x[k < cnt ? base + k : 0ull];
        }
#pragma unroll
        for (int t = 0; t < AHEAD; ++t)
            if (k0 + (uint32_t)t * S < cmax) round(k0 + (uint32_t)t * S + g.sub < cnt, key_of(px[t]));
    }
    // A chunk without an entry in the threshold's prefix bin (nearly all of them) is settled here:
    // every entry above the prefix is above the threshold, none equals it.  The others are counted
    // again once the threshold key is known.
    if (is_cand && g.sub == 0) { cb.c_gt[chunk] = n_above; cb.c_eq[chunk] = 0u; cb.rec_amb[chunk] = n_amb; }
}

// One launch for both sources of candidates: the first `hist_blocks` workgroups histogram the last
// digit of the spilled candidates (layers in SEL_CAND mode), the others run the streaming compaction
// for the layers that need it (none after a single-pass profile whose spilled range serves every
// layer: they leave after one load).  The two touch different layers.
__global__ __launch_bounds__(256, 5) void k_candidates(CompressBuffers cb, uint32_t nchunks_total, const uint32_t* chunk_big,
                                                    uint32_t hist_blocks, uint32_t ntiles, int32_t err_internal) {
    if (blockIdx.x < hist_blocks) hist3_candidates(cb, nchunks_total, chunk_big, blockIdx.x);
    else compact_tiles(cb, ntiles, err_internal, blockIdx.x - hist_blocks, gridDim.x - hist_blocks);
}

// ---------------------------------------------------------------------------------------------
// Exact threshold key and tie quota per big layer from the last-digit histogram.
__global__ __launch_bounds__(256) void k_resolve(CompressBuffers cb) {
    __shared__ uint32_t su[16];
    __shared__ uint32_t res[2];
    const uint32_t b = blockIdx.x, tid = threadIdx.x;
    const SelRec S = cb.sel[b];
    // The histogram is left at zero for the next call, whatever the mode: this kernel is its only reader.
    uint4* h4 = reinterpret_cast<uint4*>(cb.hist3 + (size_t)b * D3_BINS + tid * 16u);
    if (S.mode != SEL_PREFIX && S.mode != SEL_CAND && !(S.mode == SEL_DIRECT && S.amb != 0u)) {
        if (tid == 0) { cb.tau[b] = 0u; cb.quota[b] = 0u; }   // everything or nothing: decided by the mode alone
#pragma unroll
        for (int k = 0; k < 4; ++k) h4[k] = make_uint4(0u, 0u, 0u, 0u);
        return;
    }
    const uint32_t need = S.K - S.above;           // 1..amb entries to take from the ambiguous ones
    // thread t owns digits 16t..16t+15; we need, from the top, the digit where the running count reaches `need`
    uint32_t c[16], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint4 v = h4[k];
        c[4 * k] = v.x; c[4 * k + 1] = v.y; c[4 * k + 2] = v.z; c[4 * k + 3] = v.w;
        h4[k] = make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) sum += c[k];
    uint32_t tot;
    const uint32_t ex = block_exclusive_scan<uint32_t>(sum, su, &tot);
    // entries in digits above this thread's range
    uint32_t above = tot - ex - sum;
    if (tid == 0) { res[0] = 0xFFFFFFFFu; res[1] = 0; }
    __syncthreads();
    if (above < need && above + sum >= need) {
#pragma unroll
        for (int k = 15; k >= 0; --k) {
            if (above + c[k] >= need) { res[0] = tid * 16u + k; res[1] = need - above; break; }
            above += c[k];
        }
    }
    __syncthreads();
    if (tid == 0) {
        if (res[0] == 0xFFFFFFFFu) {               // histogram does not cover the quota (stale cache): keep all ambiguous
            cb.tau[b] = S.prefix << D2_SHIFT; cb.quota[b] = 0xFFFFFFFFu;
        } else {
            cb.tau[b] = (S.prefix << D2_SHIFT) | res[0];
            cb.quota[b] = res[1];
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Per chunk: how many candidates lie above tau and how many equal it.

// Layers served from g and h (SEL_DIRECT with a threshold): one wave per chunk with an entry in the threshold's
// prefix bin, half a chunk of loads in flight together.  Tiles in a grid-stride loop, as in the compaction.
// (Four lanes of the candidates' half of this launch read such a chunk one element at a time before: 256 dependent
// memory round trips.  Six tensors of 266 K elements in all: 59 us, now 4; ResNet-50 with two fifths of its bytes sent:
// 63 us, now 8.)
__device__ __forceinline__ void count_direct_tiles(const CompressBuffers& cb, uint32_t ntiles, uint32_t block, uint32_t nblocks) {
    if (cb.ncompact[1] == 0u) return;
    const uint32_t wave = threadIdx.x >> 6, lane = lane_id();
    const uint32_t chunks_per_tile = cb.tile_elems / CHUNK;
    for (uint32_t tile = block; tile < ntiles; tile += nblocks) {
        const LayerDesc L = cb.layers[cb.chunk_layer[tile]];
        const SelRec S = cb.sel[L.big];
        if (S.mode != SEL_DIRECT || S.amb == 0u) continue;
        const uint32_t tau = cb.tau[L.big];
        for (uint32_t cc = wave; cc < chunks_per_tile; cc += 4u) {
            const uint32_t chunk_in_layer = (tile - L.tile0) * chunks_per_tile + cc;
            if (chunk_in_layer >= L.nchunks) break;
            const uint32_t chunk = L.chunk0 + chunk_in_layer;
            uint32_t gt = cb.rec_cnt[chunk], eq = 0u;
            if (cb.rec_amb[chunk] != 0u) {       // (else every entry at or above the prefix is above tau)
                uint32_t both = 0u;              // above in the low half, equal in the high half: at most 1024 each
                // (half a chunk at a time: a whole one took this kernel past the 64 registers that eight waves a SIMD leave)
                constexpr uint32_t HALF = NQ / 2u;
#pragma unroll 1
                for (uint32_t v0 = chunk_in_layer * CHUNK; v0 < (chunk_in_layer + 1u) * CHUNK; v0 += CHUNK / 2u) {
                    QuadGH q[HALF];
                    uint32_t valid;
                    load_chunk<(int)HALF>(L, v0, q, valid);
#pragma unroll
                    for (int u = 0; u < (int)HALF; ++u)
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const uint32_t key = key_of(q[u].g[c] - q[u].h[c]);
                            const bool in = (valid >> (4 * u + c)) & 1u;
                            both += in && key > tau ? 1u : 0u;
                            both += in && key == tau ? 0x10000u : 0u;
                        }
                }
                both = wave_scan_add_u32(both);
                both = (uint32_t)__builtin_amdgcn_readlane((int)both, 63);
                gt = both & 0xFFFFu; eq = both >> 16;
            }
            if (lane == 0) { cb.c_gt[chunk] = gt; cb.c_eq[chunk] = eq; }
        }
    }
}

// Layers with candidates: four lanes per chunk.
__device__ __forceinline__ void count_candidates(const CompressBuffers& cb, uint32_t nchunks_total, const uint32_t* chunk_big,
                                                 uint32_t block) {
    constexpr uint32_t S = SUB_COUNT;
    const SubGroup g = sub_group<S>();
    const uint32_t chunk = block * (256u / S) + threadIdx.x / S;
    const bool live = chunk < nchunks_total;
    uint32_t cnt = 0, tau = 0, total = 0;
    uint64_t base = 0;
    bool settled = false;
    if (live) {
        // what the chunk index alone addresses goes out together, then the layer's record
        const uint32_t b = chunk_big[chunk], first = cb.chunk_first[chunk];
        const uint32_t amb = cb.rec_amb[chunk], start = cb.rec_start[chunk];
        total = cb.rec_cnt[chunk];
        materialise(b); materialise(first); materialise(amb); materialise(start); materialise(total);
        const SelRec S = cb.sel[b];
        const uint32_t t = cb.tau[b];
        // Only chunks with entries in the threshold's prefix bin are read again.  Of the others, those
        // of the classic pass hold nothing below the threshold prefix and pass whole; those of the
        // spilled candidates were counted by hist3_candidates.
        if ((S.mode == SEL_CAND || S.mode == SEL_PREFIX) && amb != 0u) {
            cnt = total;
            tau = t;
            base = region_start(first, b) + start;
        }
        // counted by hist3_candidates, or by the workgroups that look after the layers served from g and h
        settled = (S.mode == SEL_CAND && cnt == 0u) || S.mode == SEL_DIRECT;
    }
    uint32_t gt = 0, eq = 0;
    for (uint32_t k = g.sub; k < cnt; k += S) {
        const uint32_t key = key_of(cb.tmp_x[base + k]);
        gt += key > tau;
        eq += key == tau;
    }
#pragma unroll
    for (int d = S / 2; d > 0; d >>= 1) { gt += __shfl_xor(gt, d, 64); eq += __shfl_xor(eq, d, 64); }
    if (cnt == 0) { gt = total; eq = 0; }
    if (live && !settled && g.sub == 0) { cb.c_gt[chunk] = gt; cb.c_eq[chunk] = eq; }
}

// One launch for both, as in k_candidates; the two write the counts of different layers.
// (at least eight waves a SIMD, which the candidates' half lives by)
__global__ __launch_bounds__(256, 8) void k_chunk_count(CompressBuffers cb, uint32_t nchunks_total, const uint32_t* chunk_big,
                                                     uint32_t cand_blocks, uint32_t ntiles) {
    if (blockIdx.x < cand_blocks) count_candidates(cb, nchunks_total, chunk_big, blockIdx.x);
    else count_direct_tiles(cb, ntiles, blockIdx.x - cand_blocks, gridDim.x - cand_blocks);
}

// ---------------------------------------------------------------------------------------------
// Payload position and tie allowance of every chunk.  One workgroup per block of 1024 chunks, one
// thread per chunk.  Ties are granted to the lowest indices first, so all chunks before this
// block together keep min(their ties, quota) of them: the block's starting point follows from two
// sums over the earlier chunks of the layer, which every workgroup takes for itself (no atomics,
// no serial pass over the layer).
__device__ __forceinline__ void chunk_bases(const CompressBuffers& cb, uint32_t blk) {
    __shared__ uint32_t su[16];
    const uint32_t tid = threadIdx.x;
    const uint32_t b = cb.cblk_big[blk];
    const uint32_t li = cb.big_layer[b];
    const LayerDesc L = cb.layers[li];
    const uint32_t quota = cb.quota[b];
    const uint32_t kb = blk - L.cblk0;              // this block's number inside the layer
    uint32_t pg = 0, pe = 0;
    {
        // kb * CBLOCK is a multiple of 1024: every thread takes kb entries, sixteen loads of each table at a time (the
        // last block of the largest layer has the most to add up and sets the kernel's duration: few round trips)
        const uint32_t* pgt = cb.c_gt + L.chunk0 + tid;
        const uint32_t* peq = cb.c_eq + L.chunk0 + tid;
        for (uint32_t k = 0; k < kb; k += 16u) {
            uint32_t a[16], e[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const bool in = k + (uint32_t)u < kb;
                const size_t o = (size_t)(in ? k + (uint32_t)u : 0u) * 1024u;
                a[u] = pgt[o]; e[u] = peq[o];
                if (!in) { a[u] = 0u; e[u] = 0u; }
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) { pg += a[u]; pe += e[u]; }
        }
    }
    uint32_t gt_before, eq_before0;
    (void)block_exclusive_scan<uint32_t>(pg, su, &gt_before);
    (void)block_exclusive_scan<uint32_t>(pe, su, &eq_before0);
    const uint32_t out_before = gt_before + min(eq_before0, quota);
    const uint32_t c = kb * CBLOCK + tid;
    const bool ok = c < L.nchunks;
    const uint32_t gt = ok ? cb.c_gt[L.chunk0 + c] : 0u;
    const uint32_t eq = ok ? cb.c_eq[L.chunk0 + c] : 0u;
    const uint32_t eq_before = eq_before0 + block_exclusive_scan<uint32_t>(eq, su, nullptr);
    const uint32_t allow = eq_before < quota ? min(eq, quota - eq_before) : 0u;
    const uint32_t ob = out_before + block_exclusive_scan<uint32_t>(gt + allow, su, nullptr);
    if (ok) { cb.o_base[L.chunk0 + c] = ob; cb.o_allow[L.chunk0 + c] = allow; }
}

// ---------------------------------------------------------------------------------------------
// Write the surviving entries as payload and update the estimator.

// Layers served from g and h: one wave per chunk.  Lane l holds elements l, l + 64, ... of the chunk, so every load and
// store of a wave is one run of memory, in index order; ranks come from ballots.
// (Sixteen lanes of the candidates' half of this launch walked such a chunk in sixteen dependent rounds before: 34 us
// for six tensors of 266 K elements in all, now 6; ResNet-50 with two fifths of its bytes sent 84 us, now 59, most of
// it the candidates' half.)
__device__ __forceinline__ void finalize_direct_tiles(const CompressBuffers& cb, uint32_t ntiles, uint32_t block, uint32_t nblocks) {
    if (cb.ncompact[1] == 0u) return;
    constexpr int R = 8;                          // rows of 64 elements loaded together: sixteen loads in flight
    static_assert(CHUNK % (64u * R) == 0, "whole trips");
    const uint32_t wave = threadIdx.x >> 6, lane = lane_id();
    const uint32_t chunks_per_tile = cb.tile_elems / CHUNK;
    for (uint32_t tile = block; tile < ntiles; tile += nblocks) {
        const LayerDesc L = cb.layers[cb.chunk_layer[tile]];
        const SelRec S = cb.sel[L.big];
        if (S.mode != SEL_DIRECT) continue;
        const bool filter = S.amb != 0u;         // amb == 0: every entry is kept
        const uint32_t tau = cb.tau[L.big];
        for (uint32_t cc = wave; cc < chunks_per_tile; cc += 4u) {
            const uint32_t chunk_in_layer = (tile - L.tile0) * chunks_per_tile + cc;
            if (chunk_in_layer >= L.nchunks) break;
            const uint32_t chunk = L.chunk0 + chunk_in_layer;
            const uint32_t allow = cb.o_allow[chunk], keepn = cb.c_gt[chunk];
            if (keepn + allow == 0u) continue;
            uint32_t out_run = cb.o_base[chunk], eq_run = 0u;
#pragma unroll 1
            for (uint32_t v0 = chunk_in_layer * CHUNK; v0 < (chunk_in_layer + 1u) * CHUNK; v0 += 64u * (uint32_t)R) {
                float g[R], h[R];
#pragma unroll
                for (int t = 0; t < R; ++t) {
                    // (positions outside the layer read its entry 0, a valid address, and are dropped)
                    const uint32_t v = v0 + lane + (uint32_t)t * 64u, e = v - L.mis;
                    const uint32_t at = v >= L.mis && e < L.n ? e : 0u;
                    g[t] = gload(L.g + at); h[t] = gload(L.h + at);
                }
#pragma unroll
                for (int t = 0; t < R; ++t) {
                    const uint32_t v = v0 + lane + (uint32_t)t * 64u, e = v - L.mis;
                    const bool in = v >= L.mis && e < L.n;
                    const float x = g[t] - h[t];
                    const uint32_t key = key_of(x);
                    const bool iseq = in && filter && key == tau;
                    const uint64_t eqm = ballot(iseq);
                    const bool keep = in && (!filter || key > tau || (iseq && eq_run + mbcnt(eqm) < allow));
                    eq_run += (uint32_t)__popcll(eqm);
                    const uint64_t km = ballot(keep);
                    const uint32_t pos = out_run + mbcnt(km);
                    out_run += (uint32_t)__popcll(km);
                    if (keep && pos < S.K) {
                        const uint64_t o = S.dst + pos;
                        cb.idx_out[o] = e;
                        const float add = emit_value(cb, o, x);
                        gstore(L.h + e, h[t] + add);
                    }
                }
            }
        }
    }
}

// Layers with candidates: sixteen lanes per chunk.
__device__ __forceinline__ void finalize_candidates(const CompressBuffers& cb, uint32_t nchunks_total, const uint32_t* chunk_big,
                                                    uint32_t block) {
    const SubGroup g = sub_group();
    const uint32_t chunk = block * CHUNKS_PER_WG + threadIdx.x / SUB;
    uint32_t cnt = 0, tau = 0, allow = 0, room = 0, out_run = 0, eq_run = 0, place0 = 0;   // place0: the entry at the chunk's position 0
    uint64_t src = 0, dst = 0;
    bool filter = false;
    float* h = nullptr;
    if (chunk < nchunks_total) {
        // everything indexed by the chunk is fetched at once; one more round trip brings the layer's record
        const uint32_t b = chunk_big[chunk], first = cb.chunk_first[chunk];
        const uint32_t keepn = cb.c_gt[chunk];
        const uint32_t n_rec = cb.rec_cnt[chunk], start = cb.rec_start[chunk], amb = cb.rec_amb[chunk];
        allow = cb.o_allow[chunk];
        out_run = cb.o_base[chunk];
        materialise(b); materialise(first); materialise(keepn); materialise(n_rec); materialise(start); materialise(amb);
        materialise(allow); materialise(out_run);
        // most chunks keep nothing (the candidates are several times the payload): not read at all
        if (keepn + allow != 0u) {
            // every field of the record is valid whatever the mode; SEL_NONE and SEL_DIRECT only empty the chunk.
            // (Kept free of a nested branch on the mode: with one, the generated code left dst undefined
            // for SEL_CAND lanes.)
            const SelRec S = cb.sel[b];
            tau = cb.tau[b];
            cnt = S.mode == SEL_CAND || S.mode == SEL_PREFIX ? n_rec : 0u;
            h = S.h;
            filter = S.mode == SEL_CAND || (S.mode == SEL_PREFIX && amb != 0u);
            src = region_start(first, b) + start;
            place0 = (chunk - first) * CHUNK - S.mis;
            dst = S.dst;
            room = S.K;                            // payload slots of this layer
        }
    }
    // candidate k of the chunk
    auto fetch = [&](uint32_t k, uint32_t& idx, float& x) -> bool {
        const bool in = k < cnt;
        const uint64_t at = in ? src + k : 0ull;
        idx = place0 + cb.tmp_i[at]; x = cb.tmp_x[at];
        return in;
    };
    const uint32_t cmax = wave_max_over_groups(cnt);
    // one round: sixteen candidates of the chunk, in index order: which are kept, and where they go
    auto round = [&](bool in, float x, uint32_t& pos) -> bool {
        const uint32_t key = key_of(x);
        const bool iseq = in && filter && key == tau;
        const uint32_t eqm = ballot_sub(g, iseq);
        const bool keep = in && (!filter || key > tau || (iseq && eq_run + rank_sub(g, eqm) < allow));
        eq_run += __popc(eqm);
        const uint32_t km = ballot_sub(g, keep);
        pos = out_run + rank_sub(g, km);
        out_run += __popc(km);
        return keep && pos < room;
    };
    // A chunk rarely holds more than 64 candidates: the loads of the first four rounds go out together,
    // so the wave pays one memory round trip for them instead of four; likewise the estimator entries of what the
    // four rounds keep are read together, then written (the entries of a chunk are distinct elements).
    constexpr int AHEAD = 4;
    // (positions past the chunk's last entry read entry 0 of the buffer, a valid address, and are dropped)
    for (uint32_t k0 = 0; k0 < cmax; k0 += AHEAD * SUB) {
        uint32_t pidx[AHEAD], pos[AHEAD];
        float px[AHEAD], ph[AHEAD];
        bool pin[AHEAD], keep[AHEAD];
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) pin[t] = fetch(k0 + (uint32_t)t * SUB + g.sub, pidx[t], px[t]);
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) {
            keep[t] = false; pos[t] = 0u;
            if (k0 + (uint32_t)t * SUB < cmax) keep[t] = round(pin[t], px[t], pos[t]);
        }
        // the estimator is read here: candidates carry x and their place only
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) ph[t] = keep[t] ? gload(h + pidx[t]) : 0.0f;
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) {
            if (keep[t]) {
                const uint64_t o = dst + pos[t];
                cb.idx_out[o] = pidx[t];
                const float add = emit_value(cb, o, px[t]);
                gstore(h + pidx[t], ph[t] + add);
            }
        }
    }
}

// One launch for both, as in k_candidates; the two write different layers' payload and estimator entries.
// (at least eight waves a SIMD: with five, the Llama-shaped set's 314 us were 357)
__global__ __launch_bounds__(256, 8) void k_finalize(CompressBuffers cb, uint32_t nchunks_total, const uint32_t* chunk_big,
                                                  uint32_t cand_blocks, uint32_t ntiles) {
    if (blockIdx.x < cand_blocks) finalize_candidates(cb, nchunks_total, chunk_big, blockIdx.x);
    else finalize_direct_tiles(cb, ntiles, blockIdx.x - cand_blocks, gridDim.x - cand_blocks);
}

// ---------------------------------------------------------------------------------------------
// Small layers, one workgroup each: the layer sits in registers, eight entries a thread; the threshold key and the tie
// quota come from three histograms in LDS (11, 10 and 10 bits of the key), and the entries kept are ranked in index order
// by ballots and one scan over the 128 wave-rows.
// (Sorting the layer whole to mark its first K, then writing an index range per thread in dependent loads, took 74 us for
// a layer of 8192 entries, 40 us for 4096 and 28 us for 2048 or fewer: as long as all the other kernels of a compression.)
constexpr uint32_t SMALL_PER = SMALL_MAX / SMALL_THREADS;
__device__ __forceinline__ void small_compress(const CompressBuffers& cb, uint32_t which) {
    __shared__ uint32_t hist[2048];
    __shared__ uint32_t su[16];
    __shared__ uint32_t rows[SMALL_PER * (SMALL_THREADS / 64)];     // per (row, wave): entries above the threshold | equal << 16
    __shared__ uint32_t sh_digit, sh_need;
    __shared__ int bad;
    const uint32_t tid = threadIdx.x, wave = tid >> 6;
    const uint32_t li = cb.small_layer[which];
    const LayerDesc L = cb.layers[li];
    // the lookup kernel refuses the whole call through the status word; small layers re-check
    // their own slice so that nothing is written out of bounds
    const uint64_t K64 = cb.K[li], off = cb.offsets[li];
    if (tid == 0) bad = (*cb.status != 0);
    __syncthreads();
    if (bad || K64 == 0 || K64 > L.n || off > cb.capacity_pairs || K64 > cb.capacity_pairs - off) return;
    const uint32_t K = (uint32_t)K64;
    if (L.n <= 64u) {
        // One wave, one entry a lane: an entry's rank is how many entries go before it.  (2000 layers of 8 or 64 entries,
        // calls with some kept whole: 24 and 27 us, with the histograms 58 and 58, sorted in LDS 34 and 52.)
        if (wave != 0u) return;
        const bool in = tid < L.n;
        const float h1 = in ? gload(L.h + tid) : 0.f, x1 = in ? gload(L.g + tid) - h1 : 0.f;
        const uint32_t key = key_of(x1);
        uint32_t rank = 0u;
        for (uint32_t i = 0; i < L.n; ++i) {
            const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)key, (int)i);
            rank += other > key || (other == key && i < tid) ? 1u : 0u;
        }
        const bool keep = in && rank < K;
        const uint64_t o = off + mbcnt(ballot(keep));
        if (keep) {
            cb.idx_out[o] = tid;
            const float add = emit_value(cb, o, x1);
            gstore(L.h + tid, h1 + add);
        }
        return;
    }
    float x[SMALL_PER], h[SMALL_PER];
#pragma unroll
    for (int r = 0; r < (int)SMALL_PER; ++r) {
        const uint32_t e = tid + (uint32_t)r * SMALL_THREADS;
        x[r] = 0.f; h[r] = 0.f;
        if ((uint32_t)r * SMALL_THREADS < L.n && e < L.n) { h[r] = gload(L.h + e); x[r] = gload(L.g + e) - h[r]; }
    }
    uint32_t tau = 0u, quota = 0u;                // K == n: every entry is kept
    const bool all = K == L.n;
    if (!all) {
        uint32_t need = K;                         // entries still to take, from the top, among those sharing the digits fixed so far
        uint32_t prefix = 0u;
#pragma unroll
        for (int pass = 0; pass < 3; ++pass) {
            const uint32_t shift = pass == 0 ? 20u : pass == 1 ? 10u : 0u;
            const uint32_t mask = pass == 0 ? 2047u : 1023u;
            hist[tid] = 0u; hist[tid + 1024u] = 0u;
            __syncthreads();
#pragma unroll
            for (int r = 0; r < (int)SMALL_PER; ++r) {
                if ((uint32_t)r * SMALL_THREADS >= L.n) continue;
                const uint32_t e = tid + (uint32_t)r * SMALL_THREADS;
                const uint32_t key = key_of(x[r]);
                if (e < L.n && (pass == 0 || (key >> (pass == 1 ? 20 : 10)) == prefix)) atomicAdd(&hist[(key >> shift) & mask], 1u);
            }
            __syncthreads();
            // thread t holds bins 2t and 2t + 1
            const uint32_t c0 = hist[2u * tid], c1 = hist[2u * tid + 1u];
            uint32_t tot;
            const uint32_t ex = block_exclusive_scan<uint32_t>(c0 + c1, su, &tot);
            const uint32_t above1 = tot - ex - c0 - c1, above0 = above1 + c1;      // entries above bin 2t + 1, above bin 2t
            if (above1 < need && above1 + c1 >= need) { sh_digit = 2u * tid + 1u; sh_need = need - above1; }
            else if (above0 < need && above0 + c0 >= need) { sh_digit = 2u * tid; sh_need = need - above0; }
            __syncthreads();
            prefix = (prefix << (pass == 0 ? 0 : 10)) | sh_digit;
            need = sh_need;
            __syncthreads();
        }
        tau = prefix;
        quota = need;
    }
    // counts per (row of 1024 entries, wave), scanned in index order
    uint64_t gtm[SMALL_PER], eqm[SMALL_PER];
#pragma unroll
    for (int r = 0; r < (int)SMALL_PER; ++r) {
        const uint32_t e = tid + (uint32_t)r * SMALL_THREADS;
        const uint32_t key = key_of(x[r]);
        gtm[r] = ballot(e < L.n && (all || key > tau));
        eqm[r] = ballot(e < L.n && !all && key == tau);
        if (lane_id() == 0) rows[(uint32_t)r * (SMALL_THREADS / 64) + wave] = (uint32_t)__popcll(gtm[r]) | ((uint32_t)__popcll(eqm[r]) << 16);
    }
    __syncthreads();
    static_assert(SMALL_PER * (SMALL_THREADS / 64) == 128 && SMALL_MAX < 65536, "two counts a lane, sixteen bits each");
    if (wave == 0) {
        const uint32_t a = rows[2u * tid], b = rows[2u * tid + 1u];
        const uint32_t ex = wave_scan_add_u32(a + b) - a - b;
        rows[2u * tid] = ex;
        rows[2u * tid + 1u] = ex + a;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < (int)SMALL_PER; ++r) {
        const uint32_t e = tid + (uint32_t)r * SMALL_THREADS;
        const uint32_t at = rows[(uint32_t)r * (SMALL_THREADS / 64) + wave];
        const bool gt = (gtm[r] >> lane_id()) & 1u, eq = (eqm[r] >> lane_id()) & 1u;
        const uint32_t eq_before = (at >> 16) + mbcnt(eqm[r]);
        if (gt || (eq && eq_before < quota)) {
            const uint64_t o = off + ((at & 0xFFFFu) + mbcnt(gtm[r]) + min(eq_before, quota));
            cb.idx_out[o] = e;
            const float add = emit_value(cb, o, x[r]);
            gstore(L.h + e, h[r] + add);
        }
    }
}

__global__ __launch_bounds__(SMALL_THREADS) void k_small_compress(CompressBuffers cb) { small_compress(cb, blockIdx.x); }

// One launch for both: the blocks of chunks, and, from `nblk` on, a workgroup per small layer, which touch nothing of each
// other's (as with k_predict: on a stream of their own the small layers cost the events that bring them there and back).
__global__ __launch_bounds__(SMALL_THREADS) void k_chunk_bases(CompressBuffers cb, uint32_t nblk) {
    static_assert(SMALL_THREADS == CBLOCK, "one thread per chunk of a block");
    if (blockIdx.x < nblk) chunk_bases(cb, blockIdx.x);
    else small_compress(cb, blockIdx.x - nblk);
}

}  // namespace kimad
