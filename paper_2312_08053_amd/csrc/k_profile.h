// Error-profile kernels: two streaming histogram passes over g, h for the tiled layers, two
// per-layer scan kernels, and a whole-layer LDS sort for small layers.
//
// What they compute is the Errors matrix of the paper's Appendix C with the squared-l2 error of
// Section 3.2 (Eq. norm decomposition): E_ij = sum of x^2 over the entries TopK_{K_ij} drops.
#pragma once
#include "common.h"

namespace kimad {

// A layer that k_reduce_parts sums up: its parts (there is room for one every PK_MAX_CHUNKS chunks).
struct ReduceLayer { uint32_t big, part0, nparts, pad; };
// A workgroup's share of the streaming pass: the first chunk (it ends where the next one begins), its first part (the others follow in
// order), and the first chunk's layer, among the tiled ones and among all.
struct MainShare { uint32_t chunk, part0, big, li; };

struct ProfileBuffers {
    const LayerDesc* layers;
    const uint32_t* tile_layer;   // tile -> layer
    const uint32_t* big_layer;    // big index -> layer
    const uint32_t* small_layer;  // small index -> layer
    uint32_t tile_elems;          // elements per tile (multiple of 2048, <= 32768)
    // pass 1
    uint32_t* cnt1;               // [B][4096]
    uint64_t* sq1;                // [B][4096]
    // boundary bins
    uint8_t* lut1;                // [B][4096] digit-1 bin -> slot or NO_SLOT
    uint32_t* nslots;             // [B]
    uint32_t* slot_bin;           // [B][64]
    // pass 2
    uint32_t* cnt2;               // [B][SLOT_STRIDE][128]
    uint64_t* sq2;                // [B][SLOT_STRIDE][128]
    uint32_t* slot_cnt;           // [B][SLOT_STRIDE] totals of the slots the single pass counted itself (k_reduce_parts)
    uint64_t* slot_sq;            // [B][SLOT_STRIDE]
    // per target (layer-major, stride J)
    uint32_t* tgt_slot;           // slot, or NO_SLOT when K == n (nothing dropped)
    uint32_t* tgt_r;              // entries selected inside the boundary bin (1..count)
    uint32_t* tgt_above1;         // entries in higher digit-1 bins
    double* tgt_below;            // sum of squares of all lower digit-1 bins
    // threshold cache for the compaction pass
    uint32_t* sel_prefix;         // 19-bit prefix
    uint32_t* sel_above;          // entries with a greater prefix
    uint32_t* sel_amb;            // entries with an equal prefix
    uint32_t* diag;               // [0] uncertified entries, [1] entries fixed by the exact fallback,
                                  // [2] pool entries handed out
    // exact digit-1 histograms of the last single-pass profile: the prediction of the next one
    uint32_t* hprev;              // [B][4096]
    unsigned long long* gprev;    // [4096] their sum over the layers
    uint32_t* fresh;              // 1 while the threshold cache and the candidates describe the current g - h:
                                  // set by the profile's last kernels, cleared by the compression
    // exact fallback for entries whose bound is not tight: last-digit histograms of their prefix bins
    uint32_t* tiles_done;         // [B] tiles of a layer that a pass over its tiles is done with
    uint32_t* layer_flag;         // [B] layer has at least one pool entry
    uint32_t pool_cap;            // pool entries the plan holds: min(B * J, POOL_LIMIT)
    uint32_t* pool_prefix;        // [pool_cap]
    uint32_t* pool_big;           // [pool_cap]
    uint32_t* pool_t0;            // [pool_cap] first target (li * J + j) of the run sharing the prefix
    uint32_t* pool_cnt;           // [pool_cap] targets in that run
    uint32_t* pool_hist;          // [pool_cap][4096]
    uint32_t* tgt_unsel;          // dropped entries inside the prefix bin
    double* tgt_base;             // E without the prefix bin's share
    // fused single-pass profile
    LayerState* state;            // [B]
    const uint64_t* big_tmp0;     // [B] start of the layer's region in the candidate buffer (LayerDesc::tmp0)
    // histograms of the streaming pass, one copy ("part") per workgroup and layer, or more where a copy's counts fill up
    uint32_t* part_head;          // [nparts][PART_HEAD] whether there is one, and how its blocks were written
    unsigned long long* parts;    // [nparts][PART_STRIDE] the LDS entries, in blocks, then the exact bin-0 sum
    const MainShare* shares;      // [workgroups + 1]
    const ReduceLayer* reduce_layers;   // [B] in the order of k_reduce_parts' workgroups
    const uint32_t* chunk_big;    // chunk -> big index
    const uint32_t* chunk_first;  // chunk -> first chunk of its layer
    uint32_t nchunks_total;
    const uint32_t* swg_layer;    // sampling workgroup -> layer
    const uint32_t* swg_first;    // sampling workgroup -> its first sampled group in that layer
    uint32_t* shist;              // [B][4096] digit-1 counts of the sample
    unsigned long long* ghist;    // [4096] sample counts of all layers, scaled by the sampling stride
    uint8_t* lutc;                // [B][4096] digit-1 bin -> slot PRE_SLOTS.. filled from the candidates
    uint32_t* cursor;             // [B] candidate entries handed out so far
    uint32_t* spill_over;         // [B] a reservation did not fit the layer's region
    uint32_t* rec_start;          // per chunk: start inside the layer's candidate region
    uint32_t* rec_cnt;            // per chunk: candidates written
    // candidate buffer: x, and its position in the chunk's 1024
    float* tmp_x;
    uint16_t* tmp_i;
};

// Pool of exact last-digit histograms: one entry per (layer, threshold prefix) whose error bound is
// too wide.  A layer has at most J such prefixes, so B * J entries can never run out; plans with
// more than POOL_LIMIT of them hold POOL_LIMIT, and a candidate that finds the pool full gets NaN
// in the table (the allocation then reports a non-finite table instead of using a loose value).
constexpr uint32_t POOL_LIMIT = 65536;          // 16 KB each: at most 1 GB
constexpr uint32_t POOL_NONE = 0xFFFFFFFFu;

// ---------------------------------------------------------------------------------------------
// Pass 1: per-layer histogram of digit 1 with counts and integer sums of squares.
// One workgroup per tile; the histogram lives in LDS as packed 64-bit entries.
__global__ __launch_bounds__(256) void k_hist1(ProfileBuffers pb) {
    __shared__ unsigned long long hist[D1_BINS];
    __shared__ unsigned long long sq0;         // exact squares of bin 0 (tiny denormals)
    const uint32_t tid = threadIdx.x;
    for (uint32_t b = tid; b < D1_BINS; b += 256) hist[b] = 0ull;
    if (tid == 0) sq0 = 0ull;
    __syncthreads();

    const uint32_t tile = blockIdx.x;
    const uint32_t li = pb.tile_layer[tile];
    const LayerDesc L = pb.layers[li];
    const uint32_t vbase = (tile - L.tile0) * pb.tile_elems;
    const uint32_t iters = pb.tile_elems / 1024u;

    for (uint32_t it = 0; it < iters; it += 2) {
        Quad q[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) load_quad(L, vbase + (it + u) * 1024u + tid * 4u, q[u]);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t key = q[u].key[c];
                if (key == KEY_INVALID) continue;
                const uint32_t bin = key >> D1_SHIFT;
                if (bin != 0u) {
                    atomicAdd(&hist[bin], CNT_ONE | (unsigned long long)sq_fixed(key));
                } else {
                    atomicAdd(&hist[0], CNT_ONE);
                    if (key) atomicAdd(&sq0, sq_exact(key));
                }
            }
        }
    }
    __syncthreads();
    uint32_t* cnt = pb.cnt1 + (size_t)L.big * D1_BINS;
    unsigned long long* sq = reinterpret_cast<unsigned long long*>(pb.sq1) + (size_t)L.big * D1_BINS;
    for (uint32_t b = tid; b < D1_BINS; b += 256) {
        const unsigned long long v = hist[b];
        if (v) {
            atomicAdd(&cnt[b], (uint32_t)(v >> 48));
            const unsigned long long s = b ? (v & SQ_MASK) : sq0;
            if (s) atomicAdd(&sq[b], s);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Scan 1: per big layer, locate every candidate's boundary bin in digit 1.
// targets: K values, row `li` of a [L][J] table.
__global__ __launch_bounds__(256) void k_scan1(ProfileBuffers pb, const uint32_t* Ktab, uint32_t J) {
    __shared__ uint32_t cnt[D1_BINS];
    __shared__ uint32_t above[D1_BINS];      // entries in strictly higher bins
    __shared__ double below[D1_BINS];        // squares in strictly lower bins
    __shared__ uint32_t su[16];
    __shared__ double sd[16];
    __shared__ uint32_t tbin[MAX_SLOTS];
    __shared__ double sh_total;              // squares of the whole layer (what K = 0 drops)
    const uint32_t tid = threadIdx.x;
    const uint32_t big = blockIdx.x;
    const uint32_t li = pb.big_layer[big];
    const LayerDesc L = pb.layers[li];
    const uint32_t* gcnt = pb.cnt1 + (size_t)big * D1_BINS;
    const uint64_t* gsq = pb.sq1 + (size_t)big * D1_BINS;

    // thread t owns bins 16t .. 16t+15
    uint32_t c[16];
    double s[16];
    uint32_t csum = 0;
    double ssum = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const uint32_t b = tid * 16u + k;
        c[k] = gcnt[b];
        s[k] = sq_to_double(b, gsq[b], c[k]);
        csum += c[k];
        ssum += s[k];
    }
    uint32_t ctot;
    const uint32_t cex = block_exclusive_scan<uint32_t>(csum, su, &ctot);
    const double sex = block_exclusive_scan<double>(ssum, sd, nullptr);
    {
        uint32_t run_c = cex;      // entries in bins below the current one
        double run_s = sex;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint32_t b = tid * 16u + k;
            cnt[b] = c[k];
            below[b] = run_s;
            run_c += c[k];
            above[b] = ctot - run_c;
            run_s += s[k];
        }
        if (tid == 255u) sh_total = run_s;
    }
    uint8_t* lut = pb.lut1 + (size_t)big * D1_BINS;
    for (uint32_t b = tid; b < D1_BINS; b += 256) lut[b] = (uint8_t)NO_SLOT;
    __syncthreads();

    if (tid < J) {
        const uint32_t K = Ktab[(size_t)li * J + tid];
        uint32_t bin = 0xFFFFFFFFu;
        if (K == 0u) pb.tgt_below[(size_t)li * J + tid] = sh_total;      // nothing kept: everything is dropped
        if (K != 0u && K < L.n) {
            // smallest bin with above[bin] < K (above is non-increasing, above[4095] = 0)
            uint32_t lo = 0, hi = D1_BINS - 1;
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (above[mid] < K) hi = mid; else lo = mid + 1;
            }
            bin = lo;
            pb.tgt_r[(size_t)li * J + tid] = K - above[bin];
            pb.tgt_above1[(size_t)li * J + tid] = above[bin];
            pb.tgt_below[(size_t)li * J + tid] = below[bin];
        }
        tbin[tid] = bin;
    }
    __syncthreads();
    if (tid == 0) {
        // Targets are sorted by K, so equal boundary bins are adjacent.
        uint32_t ns = 0, last = 0xFFFFFFFFu;
        for (uint32_t j = 0; j < J; ++j) {
            const uint32_t bin = tbin[j];
            uint32_t slot = NO_SLOT;
            if (bin != 0xFFFFFFFFu) {
                if (bin != last) {
                    lut[bin] = (uint8_t)ns;
                    pb.slot_bin[(size_t)big * SLOT_STRIDE + ns] = bin;
                    last = bin;
                    ++ns;
                }
                slot = ns - 1;
            }
            pb.tgt_slot[(size_t)li * J + j] = slot;
        }
        pb.nslots[big] = ns;
        LayerState st;
        st.spill_bin = D1_BINS; st.nslots_d = ns; st.nslots_t = 0; st.redo = 1;
        st.spill_cnt = 0; st.spill_valid = 0; st.slot_lo = 0; st.run_a = 0;
        pb.state[big] = st;
    }
}

// ---------------------------------------------------------------------------------------------
// Scan 2: per big layer and candidate, locate the boundary inside digit 2, assemble E_ij and
// remember the 19-bit threshold prefix.  What is left undecided is how the `unsel` smallest of
// the `m` entries sharing that prefix split the prefix bin's exact sum of squares Q; their
// magnitudes differ by at most 2^-11 relative, and the estimate below is clamped to rigorous
// bounds.  Entries whose bound is not tight enough are counted in diag[0].
__device__ __forceinline__ float prefix_lo(uint32_t prefix) { return __uint_as_float(prefix << D2_SHIFT); }

// What comes of a candidate; the same in every lane.
struct Scan2Result {
    double E, base;
    uint32_t prefix, above, amb, unsel;
    bool flagged;
};
// One wave per candidate, of rank r in digit-1 bin `bin`, above which are above1 entries, below it squares of `below`: every
// lane holds two digit-2 bins.
__device__ __forceinline__ Scan2Result scan2_target(uint32_t lane, uint32_t bin, uint32_t r, uint32_t above1, double below, uint2 c, ulonglong2 q, double tol,
                                                    double widen) {
    // walk digit 2 from the top until r entries are covered: the boundary is the highest bin u > 0
    // with (entries above u) + cnt[u] >= r, or bin 0
    const uint32_t incl = wave_scan_add_u32(c.x + c.y);
    const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    const uint32_t above_hi = tot - incl;       // entries above bin 2*lane+1
    const uint32_t above_lo = above_hi + c.y;   // entries above bin 2*lane
    const uint64_t m_hi = ballot(above_hi + c.y >= r), m_lo = ballot(above_lo + c.x >= r);
    const int u_hi = m_hi ? 2 * (63 - __clzll((long long)m_hi)) + 1 : 0;
    const int u_lo = m_lo ? 2 * (63 - __clzll((long long)m_lo)) : 0;
    const int u = max(u_hi, u_lo);
    const int src = u >> 1;
    const uint32_t acc = (u & 1) ? __shfl(above_hi, src, 64) : __shfl(above_lo, src, 64);
    const uint32_t m = (u & 1) ? __shfl(c.y, src, 64) : __shfl(c.x, src, 64);
    const unsigned long long squ = (u & 1) ? __shfl(q.y, src, 64) : __shfl(q.x, src, 64);
    const uint32_t rsel = r - acc;              // 1..m selected inside the prefix bin
    const uint32_t unsel = m - rsel;
    double below2 = ((int)(2u * lane) < u ? sq_to_double(bin, q.x, c.x) : 0.0) +
                    ((int)(2u * lane + 1u) < u ? sq_to_double(bin, q.y, c.y) : 0.0);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) below2 += __shfl_xor(below2, d, 64);
    const uint32_t prefix = (bin << D2_BITS) | (uint32_t)u;
    double est = 0.0, half_gap = 0.0;
    if (unsel) {
        const double Q = sq_to_double(bin, squ, m);
        if ((bin >> 4) == 255u) {
            // Inf/NaN entries: the dropped ones are the lowest keys, i.e. the infinities first.
            const uint64_t nans = squ;
            const uint64_t infs = (uint64_t)m - nans;
            est = (uint64_t)unsel > infs ? __longlong_as_double(0x7FF8000000000000ll)
                                         : __longlong_as_double(0x7FF0000000000000ll);
        } else {
            // The dropped entries are the `unsel` smallest of m values in [lo, hi) whose squares sum
            // to Q: at least unsel*lo^2 and Q - rsel*hi^2, at most their mean share and unsel*hi^2.
            const double lo = (double)prefix_lo(prefix), hi = (double)prefix_lo(prefix + 1u);
            const double ub = fmin(((double)unsel / (double)m) * Q, (double)unsel * hi * hi);
            const double lb = fmin(ub, fmax((double)unsel * lo * lo, Q - (double)rsel * hi * hi));
            est = 0.5 * (lb + ub);
            half_gap = 0.5 * (ub - lb);
        }
    }
    const double base = below + below2;
    const double E = base + est;
    // single-pass slots hold midpoints of intervals 2^-23 wide (relative): part of the bound
    half_gap += E * widen;
    return {E, base, prefix, above1 + acc, m, unsel, half_gap > tol * E};
}

// One workgroup per big layer, one wave per candidate at a time.  Candidates whose error bound is
// too wide are then grouped by prefix (equal prefixes are adjacent because K ascends) and each
// group gets one pool entry for the exact last-digit pass.
// The counts may have been added by other workgroups of this launch: they are read with loads of device scope, and there
// is no fence (see k_hist2).
constexpr uint32_t SCAN2_THREADS = 768;         // (k_hist2 says why)
__device__ __forceinline__ void scan2(const ProfileBuffers& pb, uint32_t big, const uint32_t* Ktab, uint32_t J, double* err_table, double tol, double widen) {
    __shared__ uint32_t sh_prefix[KIMAD_MAX_J_CONST];
    __shared__ uint32_t sh_flag[KIMAD_MAX_J_CONST];
    __shared__ uint32_t sh_pool[KIMAD_MAX_J_CONST];     // pool entries this layer has taken
    __shared__ uint32_t sh_npool;
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                        // (else addresses are worked out ahead of the caller's loop, and kept through the counting)
    const uint32_t lane = tid & 63u;
    if (tid == 0) {
        sh_npool = 0u;
        pb.tiles_done[big] = 0u;                        // (for the exact pass; this layer's counts are complete)
    }
    const uint32_t li = pb.big_layer[big];
    constexpr uint32_t WAVES = SCAN2_THREADS / 64, PER_WAVE = (KIMAD_MAX_J_CONST + WAVES - 1u) / WAVES;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t n = pb.layers[li].n;
    // Lane u holds what there is to know of the wave's target u, and later what has come of it (four targets' fields in
    // every lane took 60 registers more, and a store per field and target).  The loads take two round trips, what a
    // target's index addresses, then what its slot addresses; the next target's bins are under way while one is worked on.
    const uint32_t jj = wave + lane * WAVES;
    const bool there = lane < PER_WAVE && jj < J;
    const size_t t = (size_t)li * J + jj;
    const uint32_t K = there ? Ktab[t] : 1u, slot = there ? pb.tgt_slot[t] : NO_SLOT;
    const uint32_t r = there ? pb.tgt_r[t] : 0u, above1 = there ? pb.tgt_above1[t] : 0u;
    const double below = there ? pb.tgt_below[t] : 0.0;
    const uint32_t bin = slot != NO_SLOT ? pb.slot_bin[(size_t)big * SLOT_STRIDE + slot] : 0u;
    uint2 c;
    ulonglong2 q;
    auto ask = [&](uint32_t u) {
        const uint32_t s = (uint32_t)__builtin_amdgcn_readlane((int)slot, (int)u);
        const size_t row = ((size_t)big * SLOT_STRIDE + (s == NO_SLOT ? 0u : s)) * D2_BINS;
        const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(pb.cnt2 + row) + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned long long* sq = reinterpret_cast<const unsigned long long*>(pb.sq2 + row) + 2u * lane;
        c = make_uint2((uint32_t)v, (uint32_t)(v >> 32));
        q = make_ulonglong2(__hip_atomic_load(sq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                            __hip_atomic_load(sq + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    };
    // (no slot: K == n or K == 0, nothing or everything is dropped)
    Scan2Result mine{K == 0u ? below : 0.0, 0.0, 0u, K == 0u ? 0u : n, 0u, 0u, false};
    uint32_t group = 0xFFFFFFFFu - jj;          // its prefix; distinct for what has none
    ask(0u);
#pragma unroll 1
    for (uint32_t u = 0; u < PER_WAVE && wave + u * WAVES < J; ++u) {
        const uint2 cu = c;
        const ulonglong2 qu = q;
        ask(min(u + 1u, PER_WAVE - 1u));
        if ((uint32_t)__builtin_amdgcn_readlane((int)slot, (int)u) == NO_SLOT) continue;
        const Scan2Result res = scan2_target(lane, (uint32_t)__builtin_amdgcn_readlane((int)bin, (int)u), (uint32_t)__builtin_amdgcn_readlane((int)r, (int)u),
                                             (uint32_t)__builtin_amdgcn_readlane((int)above1, (int)u),
                                             __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(below), (int)u),
                                                              __builtin_amdgcn_readlane(__double2loint(below), (int)u)), cu, qu, tol, widen);
        if (lane == u) { mine = res; group = res.prefix; }
    }
    if (there) {
        if (err_table) err_table[t] = mine.E;
        pb.sel_prefix[t] = mine.prefix;
        pb.sel_above[t] = mine.above;
        pb.sel_amb[t] = mine.amb;
        pb.tgt_unsel[t] = mine.unsel;
        pb.tgt_base[t] = mine.base;
    }
    if (lane < PER_WAVE && jj < KIMAD_MAX_J_CONST) { sh_prefix[jj] = group; sh_flag[jj] = err_table && mine.flagged ? 1u : 0u; }
    __syncthreads();
    if (tid < 64) {
        const uint32_t j = tid;
        const bool flagged = sh_flag[j] != 0u;
        const uint32_t prefix = sh_prefix[j];
        const uint32_t prev = __shfl_up(prefix, 1, 64);
        const bool head = j == 0 || prev != prefix;
        const uint64_t heads = ballot(head), flags = ballot(flagged);
        // run of this lane: from its head (highest head bit at or below j) to the lane before the next head
        const uint64_t below_or_eq = heads & (~0ull >> (63 - j));
        const uint32_t h0 = 63u - (uint32_t)__clzll((long long)below_or_eq);
        const uint64_t after = heads & ~((2ull << j) - 1ull);
        const uint32_t h1 = after ? (uint32_t)__ffsll((long long)after) - 1u : 64u;   // exclusive end
        const uint64_t run_mask = (h1 >= 64 ? ~0ull : ((1ull << h1) - 1ull)) & ~((1ull << h0) - 1ull);
        const bool run_flagged = (flags & run_mask) != 0;
        if (flagged) atomicAdd(&pb.diag[0], 1u);
        if (head && run_flagged && j < J) {
            const uint32_t f = atomicAdd(&pb.diag[2], 1u);
            if (f < pb.pool_cap) {
                pb.pool_prefix[f] = prefix;
                pb.pool_big[f] = big;
                pb.pool_t0[f] = li * J + j;
                pb.pool_cnt[f] = h1 - h0;
                pb.layer_flag[big] = 1u;
                sh_pool[atomicAdd(&sh_npool, 1u)] = f;
            } else {
                // pool full: no loose value leaves this call
                for (uint32_t k = h0; k < h1 && k < J; ++k)
                    err_table[(size_t)li * J + k] = __longlong_as_double(0x7FF8000000000000ll);
            }
        }
    }
    __syncthreads();
    // The pool's histograms share their memory with the streaming pass's histogram parts (dead by now): an
    // entry is cleared here, by the workgroup that takes it, before the exact pass counts into it.
    for (uint32_t k = 0; k < sh_npool; ++k)
        for (uint32_t x = tid; x < D3_BINS / 4u; x += SCAN2_THREADS)
            reinterpret_cast<uint4*>(pb.pool_hist + (size_t)sh_pool[k] * D3_BINS)[x] = make_uint4(0u, 0u, 0u, 0u);
}

// Waits until this wave's additions to memory are there for every compute unit (they are atomics of device scope, carried out
// beyond the caches: a release fence would write the caches back for nothing).
__device__ __forceinline__ void additions_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ---------------------------------------------------------------------------------------------
// Pass 2: digit-2 histograms (count + squares) of the entries that fall in a boundary bin.
// Workgroups take groups of consecutive tiles in a grid-stride loop and add their tables to the layer's once per group:
// on a small set, whose tiles are short, the additions of every tile's few thousand entries were nearly all of the pass
// (ResNet-18 with 50 ratios, 19 layers: 160 us with a flush per 4096 elements, 56 with one per 32768).
// hist2_group_tiles says how long a group is.  `gate` (optional) points at a device word that is
// zero when no layer needs this pass: the single-pass profile launches it as a fallback that
// normally has nothing to do, with a small grid that leaves after one load, and with `coarse` set
// so that the recount holds the same numbers the pass itself would have put into the slot.
//
// The scan of a layer's counts (scan2) belongs to the launch: the first `nbig` workgroups scan a layer each that has nothing to be
// counted here, and the layers that have are scanned by the workgroup that adds the last of their tiles (tiles_done), so that no
// workgroup waits for another.  A workgroup reports its layers' tiles when it is through with RUNS of them, or with all.
// Bound by the loads and LDS additions that the waves keep under way, so two workgroups share a compute unit: one clears, waits
// at its barriers or flushes while the other counts.  LDS holds two; twelve waves each leave the scan the 80 registers that it
// needs (sixteen waves leave 64: 18 of the scan's in scratch memory; with eight waves, the counting has fewer loads under way).
// Whoever finds a layer complete must not fence: a fence of device scope writes its chiplet's cache back first, and everything
// else that goes through that cache waits.
// (us by events, two launches, this one, and this one with the fence.  Nothing to count: GPT-2-shaped 19.1, 13.4, 13.4, perceptron
// 18.5, 12.6.  Recounted layers: 19 of ResNet-18 with 50 ratios 59, 57, 65, 53 of ResNet-50 82, 72, 173, 50 of the GPT-2-shaped
// set 323, 292, 456, 700 of 9 to 30 thousand entries 71, 74, 206, 169 of the Llama-shaped set 2500, 2540, 2780.  Every layer of the
// GPT-2-shaped set in the classic profile 296, 280, 503.  Sixteen waves, one workgroup to a compute unit, without the fence: GPT-2-
// shaped 352, 700 layers 90; eight waves, two: 348 and 78.  A report after four or 64 runs: the same.)
constexpr uint32_t HIST2_MAX_ELEMS = 32768;    // elements a workgroup may count before it flushes: the count field has 16 bits
// As many tiles as the counts admit, but at least 256 groups, one a compute unit, where the layers to be counted have the tiles for them.
// (Groups of 32768 elements left a perceptron of 266 K elements nine workgroups: k_hist2 9 -> 22 us, a classic profile
// 61 -> 80 us.  At least 512 or 1024 groups: 19 recounted layers of ResNet-18 56 -> 68 or 98 us, 53 of ResNet-50 72 -> 71 or 83;
// at least 128: the same as 256.)
__host__ __device__ inline uint32_t hist2_group_tiles(uint32_t ntiles, uint32_t tile_elems) {
    const uint32_t most = HIST2_MAX_ELEMS / tile_elems, share = ntiles / 256u;
    return share < 1u ? 1u : share < most ? share : most;
}
// Only tiles of layers that are to be counted are dealt out: the workgroups list these layers, whose tiles then follow one another
// (beyond LIST layers, all tiles).  (Dealt out with all others, seven layers of ResNet-18 with 50 ratios, of 9 to 37 thousand entries but for one, lay in
// a dozen workgroups, which took eight tiles each one after another, and scanned two layers in turn: 37 us, now 28 on average and 18 in a round
// with few of them.)
constexpr uint32_t HIST2_THREADS = SCAN2_THREADS;
__global__ __launch_bounds__(HIST2_THREADS, 6) void k_hist2(ProfileBuffers pb, uint32_t nbig, uint32_t ntiles, const uint32_t* gate,
                                                         uint32_t coarse, const uint32_t* Ktab, uint32_t J, double* err_table, double tol,
                                                         double widen) {
    __shared__ unsigned long long sub[MAX_SLOTS * D2_BINS];   // 64 KB
    __shared__ unsigned long long sub0[D2_BINS];              // exact squares when the slot is bin 0
    __shared__ uint8_t lut[D1_BINS];
    constexpr uint32_t RUNS = 8, LIST = HIST2_THREADS;
    __shared__ uint32_t run_big[RUNS], run_tiles[RUNS];       // tiles counted and not yet reported, by layer
    __shared__ uint64_t sh_which;
    __shared__ uint32_t tile_end[1024], su[16];               // tiles up to a listed layer's last; behind them the greatest number
    __shared__ uint16_t listed[LIST];                         // the layer, counted from the list's first
    uint32_t tid = threadIdx.x;
    const bool counting = blockIdx.x >= nbig;
    if (counting && gate && *gate == 0u) return;
    if (tid == 0) run_big[0] = blockIdx.x;      // (the layer of one that only scans)
    // with up to LIST layers, those that are to be counted
    const bool list = nbig <= LIST;
    if (counting && list) {
        uint32_t mine = 0u, n;
        if (tid < nbig) {
            const LayerState st = pb.state[tid];
            if (st.redo && st.nslots_d != 0u) mine = pb.layers[pb.big_layer[tid]].ntiles;
        }
        for (uint32_t x = tid; x < 1024u; x += HIST2_THREADS) tile_end[x] = 0xFFFFFFFFu;
        const uint64_t has = ballot(mine != 0u);
        const uint32_t before = block_exclusive_scan<uint32_t>(mine, su, &n);                            // (has barriers)
        const uint32_t at = block_exclusive_scan<uint32_t>((tid & 63u) == 0u ? (uint32_t)__popcll(has) : 0u, su, nullptr);
        const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        if (mine) { tile_end[first + mbcnt(has)] = before + mine; listed[first + mbcnt(has)] = (uint16_t)tid; }
        ntiles = (uint32_t)__builtin_amdgcn_readfirstlane((int)n);
        __syncthreads();
    }
    const uint32_t group_tiles = hist2_group_tiles(ntiles, pb.tile_elems);
    uint32_t tile0 = (blockIdx.x - nbig) * group_tiles, tile = tile0;        // the group, and its next tile
    for (;;) {
    uint32_t runs = 0u;
    while (counting && runs < RUNS && tile0 < ntiles) {
    asm volatile("" : "+v"(tid));               // (else addresses are worked out ahead of the loop, and kept through the scan)
    // the group's tiles of one layer
    uint32_t li, end;                           // the layer, and the tile behind its last
    if (list) {
        uint32_t at = 0u;
        for (uint32_t half = 512u; half; half >>= 1)
            if ((uint32_t)__builtin_amdgcn_readfirstlane((int)tile_end[at + half - 1u]) <= tile) at += half;
        end = (uint32_t)__builtin_amdgcn_readfirstlane((int)tile_end[at]);
        li = pb.big_layer[__builtin_amdgcn_readfirstlane((int)listed[at])];
    } else {
        li = pb.tile_layer[tile];
        end = pb.layers[li].tile0 + pb.layers[li].ntiles;
    }
    const LayerDesc L = pb.layers[li];
    const LayerState st = pb.state[L.big];
    const uint32_t ns = st.nslots_d;
    const uint32_t last = min(min(ntiles, tile0 + group_tiles), end), first = L.ntiles - (end - tile), count = last - tile;      // (first: in the layer)
    tile = last;
    if (tile == min(ntiles, tile0 + group_tiles)) { tile0 += (gridDim.x - nbig) * group_tiles; tile = tile0; }
    if (!st.redo || ns == 0) continue;
    {
        const uint32_t* src = reinterpret_cast<const uint32_t*>(pb.lut1 + (size_t)L.big * D1_BINS);
        uint32_t* dst = reinterpret_cast<uint32_t*>(lut);
        for (uint32_t b = tid; b < D1_BINS / 4; b += HIST2_THREADS) dst[b] = src[b];
    }
    for (uint32_t b = tid; b < ns * D2_BINS; b += HIST2_THREADS) sub[b] = 0ull;
    if (tid < D2_BINS) sub0[tid] = 0ull;
    __syncthreads();

    const uint32_t vend = (first + count) * pb.tile_elems;
    const uint32_t lane4 = 4u * (tid & 63u);
    constexpr uint32_t QUADS = 2;               // a thread's loads under way
    for (uint32_t v = first * pb.tile_elems + (uint32_t)__builtin_amdgcn_readfirstlane(tid & ~63u) * 4u; v < vend;
         v += 4u * QUADS * HIST2_THREADS) {
        Quad q[QUADS];
#pragma unroll
        for (uint32_t u = 0; u < QUADS; ++u) {
            if (v + u * 4u * HIST2_THREADS < vend) load_quad(L, v + u * 4u * HIST2_THREADS + lane4, q[u]);
            else { q[u].key[0] = q[u].key[1] = q[u].key[2] = q[u].key[3] = KEY_INVALID; }
        }
#pragma unroll
        for (uint32_t u = 0; u < QUADS; ++u) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t key = q[u].key[c];
                if (key == KEY_INVALID) continue;
                const uint32_t bin = key >> D1_SHIFT;
                const uint32_t slot = lut[bin];
                if (slot == NO_SLOT) continue;
                const uint32_t d2 = (key >> D2_SHIFT) & (D2_BINS - 1);
                if (bin != 0u) {
                    atomicAdd(&sub[slot * D2_BINS + d2],
                              CNT_ONE | (unsigned long long)(coarse ? sq_coarse(key) : sq_fixed(key)));
                } else {
                    atomicAdd(&sub[slot * D2_BINS + d2], CNT_ONE);
                    if (key) atomicAdd(&sub0[d2], sq_exact(key));
                }
            }
        }
    }
    __syncthreads();
    uint32_t* cnt = pb.cnt2 + (size_t)L.big * SLOT_STRIDE * D2_BINS;
    unsigned long long* sq = reinterpret_cast<unsigned long long*>(pb.sq2) + (size_t)L.big * SLOT_STRIDE * D2_BINS;
    const uint32_t slot0 = lut[0];   // slot of bin 0, if it is a boundary bin
    for (uint32_t b = tid; b < ns * D2_BINS; b += HIST2_THREADS) {
        const unsigned long long v = sub[b];
        if (v) {
            atomicAdd(&cnt[b], (uint32_t)(v >> 48));
            const unsigned long long s = (b / D2_BINS == slot0) ? sub0[b % D2_BINS] : (v & SQ_MASK);
            if (s) atomicAdd(&sq[b], s);
        }
    }
    if (tid == 0) { run_big[runs] = (uint32_t)L.big; run_tiles[runs] = count; }
    ++runs;
    __syncthreads();                            // the next tiles reuse the LDS tables
    }
    // which of the runs' layers are scanned here
    if (counting) {
        if (runs == 0u) return;
        additions_done();
        __syncthreads();
        if (tid < 64u) {
            const uint32_t b = tid < runs ? run_big[tid] : 0u;
            const bool last = tid < runs && atomicAdd(&pb.tiles_done[b], run_tiles[tid]) + run_tiles[tid] == pb.layers[pb.big_layer[b]].ntiles;
            const uint64_t which = ballot(last);
            if (tid == 0) sh_which = which;
        }
    } else if (tid == 0) {
        const LayerState st = pb.state[blockIdx.x];
        sh_which = !st.redo || st.nslots_d == 0u ? 1ull : 0ull;
    }
    __syncthreads();
    uint64_t which = sh_which;
    while (which) {
        scan2(pb, (uint32_t)__builtin_amdgcn_readfirstlane(run_big[__builtin_ctzll(which)]), Ktab, J, err_table, tol, widen);
        __syncthreads();
        which &= which - 1ull;
    }
    if (!counting || tile0 >= ntiles) return;
    }
}

// Exact fallback, scan of a pool entry by one wave.  With the full key known, the squares of the
// `unsel` smallest entries of the prefix bin are summed exactly in fp64, smallest first.
// A quarter of the digits at a time goes through `stage`, the wave's part of LDS: read from memory in whole lines, summed up
// sixteen neighbouring digits a lane.  (Four words of them lie at a place that a lane's number moves, so that sixteen lanes'
// reads fall on all banks.  Entries that need this are ties as a rule, so most digits are empty, and passed over.)
constexpr uint32_t SCAN3_WORDS = D3_BINS / 4u;
__device__ __forceinline__ void scan_pool_entry(const ProfileBuffers& pb, uint32_t f, double* err_table, uint32_t* stage) {
    constexpr uint32_t QUARTERS = 4, PAIRS = SCAN3_WORDS / 128u;
    static_assert(SCAN3_WORDS == 64u * 16u, "sixteen digits a lane");
    const uint32_t lane = lane_id();
    const uint32_t prefix = pb.pool_prefix[f], t0 = pb.pool_t0[f], targets = pb.pool_cnt[f];
    const uint32_t my_unsel = lane < targets ? pb.tgt_unsel[t0 + lane] : 0u;
    const double my_base = lane < targets ? pb.tgt_base[t0 + lane] : 0.0;
    const uint32_t* h = pb.pool_hist + (size_t)f * D3_BINS;
    auto square = [&](uint32_t d3) {
        const double v = (double)__uint_as_float((prefix << D2_SHIFT) | d3);
        return v * v;
    };
    unsigned long long v[PAIRS];
    auto ask = [&](uint32_t q) {
#pragma unroll
        for (uint32_t i = 0; i < PAIRS; ++i)
            v[i] = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(h + q * SCAN3_WORDS) + i * 64u + lane, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
    };
    uint32_t cex[QUARTERS], ctot = 0u;          // entries in digits below the lane's, their squares
    double sex[QUARTERS], stot = 0.0;
    ask(0u);
#pragma unroll
    for (uint32_t q = 0; q < QUARTERS; ++q) {
        wave_sync_lds();
#pragma unroll
        for (uint32_t i = 0; i < PAIRS; ++i) {
            const uint32_t owner = 8u * i + lane / 8u, four = (lane / 2u) & 3u;
            *reinterpret_cast<unsigned long long*>(stage + 16u * owner + 4u * (four ^ ((owner >> 2) & 3u)) + 2u * (lane & 1u)) = v[i];
        }
        if (q + 1u < QUARTERS) ask(q + 1u);
        wave_sync_lds();
        uint32_t csum = 0u;
        double ssum = 0.0;
#pragma unroll
        for (uint32_t four = 0; four < 4u; ++four) {
            const uint4 c = *reinterpret_cast<const uint4*>(stage + 16u * lane + 4u * (four ^ ((lane >> 2) & 3u)));
            const uint32_t d3 = q * SCAN3_WORDS + 16u * lane + 4u * four;
            const uint32_t sum = c.x + c.y + c.z + c.w;
            if (ballot(sum != 0u) == 0ull) continue;
            csum += sum;
            ssum += (double)c.x * square(d3);
            ssum += (double)c.y * square(d3 + 1u);
            ssum += (double)c.z * square(d3 + 2u);
            ssum += (double)c.w * square(d3 + 3u);
        }
        cex[q] = ctot;
        sex[q] = stot;
        if (ballot(csum != 0u) == 0ull) continue;
        const uint32_t ci = wave_scan_add_u32(csum);
        const double si = wave_inclusive_scan<double>(ssum), before = __shfl_up(si, 1, 64);
        cex[q] += ci - csum;
        if (lane) sex[q] += before;
        ctot += (uint32_t)__builtin_amdgcn_readlane((int)ci, 63);
        stot += __shfl(si, 63, 64);
    }
    for (uint32_t k = 0; k < targets; ++k) {
        const uint32_t unsel = (uint32_t)__builtin_amdgcn_readlane((int)my_unsel, (int)k);
        double U = 0.0;
        if (unsel) {
            // the last lane with fewer than `unsel` entries below its digits, then the last such digit: all below it are dropped whole
            uint32_t quarter = 0u, owner = 0u, below = 0u;
#pragma unroll
            for (uint32_t q = 0; q < QUARTERS; ++q) {
                const uint64_t fewer = ballot(cex[q] < unsel);
                if (!fewer) continue;
                quarter = q;
                owner = 63u - (uint32_t)__clzll((long long)fewer);
                below = (uint32_t)__builtin_amdgcn_readlane((int)cex[q], (int)owner);
                U = __shfl(sex[q], (int)owner, 64);
            }
            const uint32_t d0 = quarter * SCAN3_WORDS + 16u * owner;
            const uint32_t c = __hip_atomic_load(h + d0 + (lane & 15u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            uint32_t d = 0u;
            for (; d < 15u; ++d) {
                const uint32_t cd = (uint32_t)__builtin_amdgcn_readlane((int)c, (int)d);
                if (below + cd >= unsel) break;
                below += cd;
                U += (double)cd * square(d0 + d);
            }
            U += (double)(unsel - below) * square(d0 + d);
        }
        if (lane == k) err_table[t0 + k] = my_base + U;
    }
    if (lane == 0) atomicAdd(&pb.diag[1], targets);
}

// Exact fallback: last-digit histogram of every pooled prefix bin.  One workgroup per tile; tiles of layers without pool
// entries return at once.  A layer's entries are scanned by the workgroup that counts the last of its tiles, a wave an
// entry, so that no workgroup waits for another.  The counting is bound by the loads and additions to memory under way,
// so the scan is kept to what leaves a SIMD eight waves (64 registers; 4 KB of LDS a wave); sixteen waves take a layer's entries,
// 64 at most, in four turns.
// (us by events, as two launches, with a scan by whole workgroups of 256 threads one entry after another, and now.  No entries, as
// a rule: 12.3, 6.0, 6.0.  About 30 entries a layer: one of 20 thousand 33, 190, 27; of 1 M 318, 473, 320; a perceptron's two 78,
// 283, 78; 700 of 9 to 30 thousand 1080, 2900, 810; ResNet-50's 2100, 2750, 2050; 50 of the GPT-2-shaped set 14400, 14700, 13500.
// 512 threads: the same but for 1 M 329, a perceptron 91.  At most 512 or 2048 workgroups: GPT-2-shaped 14100 and 13900.)
constexpr uint32_t HIST3_THREADS = 1024;
__global__ __launch_bounds__(HIST3_THREADS, 8) void k_hist3p(ProfileBuffers pb, uint32_t ntiles, double* err_table, uint32_t mark_fresh) {
    __shared__ uint32_t pfx[KIMAD_MAX_J_CONST];   // a layer has at most J pooled prefixes
    __shared__ uint32_t pid[KIMAD_MAX_J_CONST];
    __shared__ uint32_t npool, sh_last;
    __shared__ __align__(16) uint32_t stage[HIST3_THREADS / 64u][SCAN3_WORDS];
    const uint32_t tid = threadIdx.x, lane4 = 4u * lane_id();
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    if (blockIdx.x == 0 && tid == 0 && mark_fresh) *pb.fresh = 1u;     // the grid profile's last kernel on the caller's stream
    if (pb.diag[2] == 0u) return;               // no pool entries at all: the usual case
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint32_t li = pb.tile_layer[tile];
    const LayerDesc L = pb.layers[li];
    if (!pb.layer_flag[L.big]) continue;
    __syncthreads();                            // the previous tile's readers are done with the lists
    if (tid == 0) npool = 0;
    __syncthreads();
    const uint32_t total = min(pb.diag[2], pb.pool_cap);
    for (uint32_t f = tid; f < total; f += HIST3_THREADS) {
        if (pb.pool_big[f] == (uint32_t)L.big) {
            const uint32_t k = atomicAdd(&npool, 1u);
            if (k < KIMAD_MAX_J_CONST) { pfx[k] = pb.pool_prefix[f]; pid[k] = f; }
        }
    }
    __syncthreads();
    const uint32_t np = min(npool, (uint32_t)KIMAD_MAX_J_CONST);
    const uint32_t vbase = (tile - L.tile0) * pb.tile_elems;
    for (uint32_t v = 256u * wave; v < pb.tile_elems; v += 4u * HIST3_THREADS) {
        Quad q;
        load_quad(L, vbase + v + lane4, q);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t key = q.key[c];
            uint32_t f = POOL_NONE;
            if (key != KEY_INVALID) {
                const uint32_t p = key >> D2_SHIFT;
                for (uint32_t k = 0; k < np; ++k) if (pfx[k] == p) f = pid[k];
            }
            const bool a = f != POOL_NONE;
            const uint64_t am = ballot(a);
            if (am == 0) continue;
            // one atomic per wave when all matching lanes hold the same key (constants, zeros)
            const uint32_t first_lane = (uint32_t)__ffsll((long long)am) - 1u;
            const uint32_t k0 = __shfl(key, first_lane, 64);
            if (ballot(a && key != k0) == 0) {
                if (lane_id() == first_lane) atomicAdd(&pb.pool_hist[(size_t)f * D3_BINS + (key & (D3_BINS - 1))], (uint32_t)__popcll(am));
            } else if (a) {
                atomicAdd(&pb.pool_hist[(size_t)f * D3_BINS + (key & (D3_BINS - 1))], 1u);
            }
        }
    }
    additions_done();                           // before the tile counts as done
    __syncthreads();
    if (tid == 0) sh_last = atomicAdd(&pb.tiles_done[L.big], 1u) + 1u == L.ntiles ? 1u : 0u;
    __syncthreads();
    if (sh_last)
        for (uint32_t k = wave; k < np; k += HIST3_THREADS / 64u) scan_pool_entry(pb, (uint32_t)__builtin_amdgcn_readfirstlane(pid[k]), err_table, stage[wave]);
    }
}

// ---------------------------------------------------------------------------------------------
// Small layers: the magnitudes of the whole layer are sorted, largest first, by one workgroup; E_ij is the suffix sum
// of squares in that order, in fp64.
constexpr uint32_t SMALL_THREADS = 1024;
constexpr uint32_t SORT_PER = SMALL_MAX / SMALL_THREADS;     // 8 values a thread
static_assert(SORT_PER == 8, "the sort below is written for eight values a thread");

// The value the lane `X` away (lane index xor X) holds, X = 1, 2, 4, 8, 16, 32.
template <int X>
__device__ __forceinline__ uint32_t lane_xor_u32(uint32_t v) {
    if (X == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);      // quad_perm [1,0,3,2]
    if (X == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);      // quad_perm [2,3,0,1]
    if (X == 4) {                                                                                    // reversed quads, then reversed eights
        const int q = __builtin_amdgcn_update_dpp(0, (int)v, 0x1B, 0xF, 0xF, false);
        return (uint32_t)__builtin_amdgcn_update_dpp(0, q, 0x141, 0xF, 0xF, false);
    }
    if (X == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, false);     // row_ror:8
    return __shfl_xor(v, X, 64);
}

// The smaller of two values where `k` is 0, the larger where it is ~0: one instruction for either direction.
__device__ __forceinline__ uint32_t min_or_max(uint32_t a, uint32_t b, uint32_t k) {
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(k));
    return r;
}
// Compare-exchange of every value with the lane X away: the lane whose bit X is clear keeps the smaller if `up`.
template <int X>
__device__ __forceinline__ void sort_lanes(uint32_t (&v)[SORT_PER], bool up) {
    const uint32_t k = ((lane_id() & (uint32_t)X) == 0u) == up ? 0u : ~0u;
#pragma unroll
    for (int r = 0; r < (int)SORT_PER; ++r) {
        if constexpr (X >= 16) {
            // (both lanes of a pair get both values)
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            const u32x2 p = X == 16 ? __builtin_amdgcn_permlane16_swap(v[r], v[r], false, false) : __builtin_amdgcn_permlane32_swap(v[r], v[r], false, false);
            v[r] = min_or_max(p.x, p.y, k);
        } else {
            v[r] = min_or_max(v[r], lane_xor_u32<X>(v[r]), k);
        }
    }
}
// The same among a thread's own values, distance D = 1, 2, 4; K: the run length being merged if it is inside a thread
// (2, 4: the direction then alternates among its values), else 8 and `up` holds for all of them.
template <int D, int K>
__device__ __forceinline__ void sort_own(uint32_t (&v)[SORT_PER], bool up) {
    const uint32_t k = up ? 0u : ~0u;
#pragma unroll
    for (int r = 0; r < (int)SORT_PER; ++r) {
        if (r & D) continue;
        const uint32_t a = v[r], b = v[r + D];
        if (K < 8) {
            v[r] = (r & K) == 0 ? min(a, b) : max(a, b);
            v[r + D] = (r & K) == 0 ? max(a, b) : min(a, b);
        } else {
            v[r] = min_or_max(a, b, k);
            v[r + D] = min_or_max(a, b, ~k);
        }
    }
}

// Bitonic sort, ascending, of P values (a power of two, 8 to SMALL_MAX): value 8 t + r is v[r] of thread t; threads
// from P / 8 on take part in the barriers only.  The result is left in `a` (P words), behind a barrier.  Distances below
// 8 are inside a thread, below 512 inside a wave (DPP moves, lane swaps for the two widest), and only the ten steps of the
// largest layer that cross waves go through LDS.  Sorting (magnitude, index) pairs of 64 bits through LDS at every
// step, as before, took 65 to 79 us of k_small_profile on a layer of 8192 entries and 40 us on one of 4096; the order
// among equal magnitudes changes no sum.
__device__ __forceinline__ void sort_small(uint32_t (&v)[SORT_PER], uint32_t* a, uint32_t P) {
    const uint32_t tid = threadIdx.x, base = tid * SORT_PER;
    const bool mine = base < P;                  // (wave-uniform from P = 512 on; below, one wave holds everything)
    const bool wave_mine = (tid & ~63u) * SORT_PER < P;
    // (Waves without values would take issue slots from those that sort: 2000 layers of 500 entries 76 us, now 43; 67 when
    // the pairs were sorted through LDS.)
    if (wave_mine) {
        sort_own<1, 2>(v, true);
        sort_own<2, 4>(v, true);
        sort_own<1, 4>(v, true);
    }
    for (uint32_t k = 8; k <= P; k <<= 1) {
        const bool up = (base & k) == 0u;
        for (uint32_t d = k >> 1; d >= 512u; d >>= 1) {
            if (mine) {
                uint4* at = reinterpret_cast<uint4*>(a + base);
                at[0] = make_uint4(v[0], v[1], v[2], v[3]);
                at[1] = make_uint4(v[4], v[5], v[6], v[7]);
            }
            __syncthreads();
            if (mine) {
                const uint4* from = reinterpret_cast<const uint4*>(a + (base ^ d));
                const uint4 o0 = from[0], o1 = from[1];
                const uint32_t o[SORT_PER] = {o0.x, o0.y, o0.z, o0.w, o1.x, o1.y, o1.z, o1.w};
                const uint32_t keep = ((base & d) == 0u) == up ? 0u : ~0u;
#pragma unroll
                for (int r = 0; r < (int)SORT_PER; ++r) v[r] = min_or_max(v[r], o[r], keep);
            }
            __syncthreads();
        }
        if (!wave_mine) continue;
        if (k >= 512u) sort_lanes<32>(v, up);
        if (k >= 256u) sort_lanes<16>(v, up);
        if (k >= 128u) sort_lanes<8>(v, up);
        if (k >= 64u) sort_lanes<4>(v, up);
        if (k >= 32u) sort_lanes<2>(v, up);
        if (k >= 16u) sort_lanes<1>(v, up);
        sort_own<4, 8>(v, up);
        sort_own<2, 8>(v, up);
        sort_own<1, 8>(v, up);
    }
    if (mine) {
        uint4* at = reinterpret_cast<uint4*>(a + base);
        at[0] = make_uint4(v[0], v[1], v[2], v[3]);
        at[1] = make_uint4(v[4], v[5], v[6], v[7]);
    }
    __syncthreads();
}

__device__ __forceinline__ uint32_t next_pow2(uint32_t n) {
    uint32_t p = 1;
    while (p < n) p <<= 1;
    return p;
}

__device__ __forceinline__ void small_profile(const ProfileBuffers& pb, uint32_t which, const uint32_t* Ktab, uint32_t J, double* err_table) {
    __shared__ __align__(16) uint32_t a[SMALL_MAX];   // 32 KB: 0x7fffffff - key, ascending
    __shared__ double loc[SMALL_THREADS];             // per-thread sums, then exclusive suffix sums
    __shared__ double sd[16];
    const uint32_t li = pb.small_layer[which];
    const LayerDesc L = pb.layers[li];
    const uint32_t P = next_pow2(L.n < SORT_PER ? SORT_PER : L.n);
    {
        uint32_t v[SORT_PER];
        // coalesced loads, all in flight together; which thread holds which value does not matter to the sort
#pragma unroll
        for (int r = 0; r < (int)SORT_PER; ++r) {
            const uint32_t e = threadIdx.x + (uint32_t)r * SMALL_THREADS;
            v[r] = 0xFFFFFFFFu;
            if ((uint32_t)r * SMALL_THREADS < L.n && e < L.n) v[r] = 0x7FFFFFFFu - key_of(gload(L.g + e) - gload(L.h + e));
        }
        if (P < SMALL_MAX) {
            // a shorter layer's values lie with the first rows of threads: hand every thread below P / 8 its eight
#pragma unroll
            for (int r = 0; r < (int)SORT_PER; ++r) {
                const uint32_t e = threadIdx.x + (uint32_t)r * SMALL_THREADS;
                if ((uint32_t)r * SMALL_THREADS < P && e < P) a[e] = v[r];
            }
            __syncthreads();
            if (threadIdx.x * SORT_PER < P) {
                const uint4* from = reinterpret_cast<const uint4*>(a + threadIdx.x * SORT_PER);      // (P is a multiple of eight)
                const uint4 v0 = from[0], v1 = from[1];
                v[0] = v0.x; v[1] = v0.y; v[2] = v0.z; v[3] = v0.w; v[4] = v1.x; v[5] = v1.y; v[6] = v1.z; v[7] = v1.w;
            }
            __syncthreads();
        }
        sort_small(v, a, P);
    }
    // thread t owns ranks [t*per, (t+1)*per) and sums their squares from the smallest upward
    const uint32_t per = P / SMALL_THREADS ? P / SMALL_THREADS : 1u;
    const uint32_t tid = threadIdx.x;
    double local = 0.0;
    for (uint32_t k = per; k-- > 0;) {
        const uint32_t rk = tid * per + k;
        if (rk < L.n) {
            const uint32_t key = 0x7FFFFFFFu - a[rk];
            const double v = (double)__uint_as_float(key);
            local += v * v;
        }
    }
    loc[tid] = local;
    __syncthreads();
    // exclusive suffix over threads: scan the per-thread sums in reversed thread order
    const double rv = loc[SMALL_THREADS - 1u - tid];
    const double ex = block_exclusive_scan<double>(rv, sd, nullptr);
    __syncthreads();
    loc[SMALL_THREADS - 1u - tid] = ex;               // sum of the squares owned by all later threads
    __syncthreads();
    if (tid < J) {
        const uint32_t K = Ktab[(size_t)li * J + tid];
        double E = 0.0;
        if (K < L.n) {
            // ranks >= K are dropped: everything owned by later threads, then the tail of K's owner
            const uint32_t owner = K / per;
            E = loc[owner];
            for (uint32_t rk = (owner + 1) * per; rk-- > K;) {
                if (rk < L.n) {
                    const uint32_t key = 0x7FFFFFFFu - a[rk];
                    const double v = (double)__uint_as_float(key);
                    E += v * v;
                }
            }
        }
        err_table[(size_t)li * J + tid] = E;
    }
}

__global__ __launch_bounds__(SMALL_THREADS) void k_small_profile(ProfileBuffers pb, const uint32_t* Ktab, uint32_t J,
                                                                 double* err_table, uint32_t mark_fresh) {
    if (blockIdx.x == 0 && threadIdx.x == 0 && mark_fresh) *pb.fresh = 1u;   // (plans without tiled layers have no other profile kernel)
    small_profile(pb, blockIdx.x, Ktab, J, err_table);
}

}  // namespace kimad
