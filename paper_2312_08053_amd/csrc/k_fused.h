// Single-pass error profile.
//
// The classic profile (k_profile.h) reads g and h twice: once to find every candidate's boundary
// bin in digit 1, once to histogram digit 2 inside those bins.  Here a sampling pre-pass over
// ~1/16 of each layer (a plan's first profile; later ones use the exact digit-1 histogram the previous
// profile left: successive gradients of a layer are distributed alike) predicts, per layer,
//   * which digit-1 bins can hold the boundary of a "dense" candidate (K beyond the top few
//     percent): those bins get digit-2 slots before the pass, and
//   * a spill bin: every entry at or above it (the top few percent, sized from the budget hint)
//     is written to the candidate buffer, x and its place in the chunk, in index order inside each chunk.
// One streaming pass then builds the exact digit-1 histogram, the digit-2 histograms of the
// predicted bins and the candidate buffer.  Candidates whose boundary lies in the spilled range
// get their digit-2 histograms from the candidate buffer (a few percent of the data), and the
// compaction later selects from the candidates instead of reading g and h again.
//
// Nothing in the result depends on the prediction: a boundary that falls outside what was
// predicted marks the layer for a recount by the classic full pass (LayerState::redo), and a
// chosen K beyond the spilled range makes the compaction read g and h for that layer.
//
// Computes the same quantities as k_profile.h: the Errors matrix of the paper's Appendix C with
// the squared-l2 error of Section 3.2.
#pragma once
#include "common.h"
#include "k_profile.h"

namespace kimad {

constexpr uint32_t SAMPLE_GROUPS_PER_WG = 48;   // sampled chunks one sampling workgroup reads: three per wave (every
                                                // workgroup ends with a flush of its histogram through global
                                                // atomics, which is what the kernel's time is made of: fewer, longer
                                                // workgroups were faster at every size tried, 4 to 48)
constexpr uint32_t FUSED_THREADS = 1024;
constexpr uint32_t FUSED_WAVES = FUSED_THREADS / 64;

__device__ __forceinline__ uint32_t hash32(uint32_t a) {
    a ^= a >> 16; a *= 0x7feb352du; a ^= a >> 15; a *= 0x846ca68bu; a ^= a >> 16;
    return a;
}

// Chunk of the layer read by sampled group `gidx`: one per `stride` chunks, at a hashed phase.
__device__ __forceinline__ uint32_t sampled_chunk(uint32_t gidx, uint32_t stride) {
    return gidx * stride + (stride > 1 ? hash32(gidx * 2654435761u + 12345u) % stride : 0u);
}

// ---------------------------------------------------------------------------------------------
// Sampling pre-pass: digit-1 counts of the sampled chunks.
// One wave per sampled chunk: all of a workgroup's loads are in flight together.
constexpr uint32_t SAMPLE_THREADS = 1024;
__global__ __launch_bounds__(SAMPLE_THREADS) void k_sample(ProfileBuffers pb) {
    __shared__ uint32_t hist[D1_BINS];
    const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
    for (uint32_t b = tid; b < D1_BINS; b += SAMPLE_THREADS) hist[b] = 0u;
    __syncthreads();
    const uint32_t li = pb.swg_layer[blockIdx.x];
    const LayerDesc L = pb.layers[li];
    const uint32_t first = pb.swg_first[blockIdx.x];
    for (uint32_t k = wave; k < SAMPLE_GROUPS_PER_WG; k += SAMPLE_THREADS / 64) {
        const uint32_t chunk = sampled_chunk(first + k, L.sstride);
        if (chunk >= L.nchunks) continue;
        const uint32_t vbase = chunk * CHUNK;
        Quad q[NQ];
#pragma unroll
        for (int u = 0; u < (int)NQ; ++u) load_quad(L, vbase + u * 256u + lane * 4u, q[u]);
#pragma unroll
        for (int u = 0; u < (int)NQ; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (q[u].key[c] != KEY_INVALID) atomicAdd(&hist[q[u].key[c] >> D1_SHIFT], 1u);
    }
    __syncthreads();
    uint32_t* sh = pb.shist + (size_t)L.big * D1_BINS;
    for (uint32_t b = tid; b < D1_BINS; b += SAMPLE_THREADS) {
        const uint32_t v = hist[b];
        if (v) {
            atomicAdd(&sh[b], v);
            atomicAdd(&pb.ghist[b], (unsigned long long)v * L.sstride);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Prediction: per big layer, the spill bin and the digit-1 bins that get a slot.
// `budget_pairs` = expected budget of the following allocation in pairs (0 = unknown); `unit_pairs` = pairs of one cost
// unit of that allocation.
// `counts` / `gcounts`: per layer and summed digit-1 counts to predict from: the sample of k_sample (scaled to the
// population through the layer's size), or the exact histogram of the previous profile on this plan (successive
// gradients of a layer are distributed alike; a layer whose boundary bins moved is recounted like any other
// misprediction).  `fold_zero`: also clear what a profile must find at zero (no separate clearing launch).
constexpr uint32_t PREDICT_THREADS = 256;
__device__ __forceinline__ void predict(const ProfileBuffers& pb, uint32_t big, uint32_t nbig, const uint32_t* Ktab, uint32_t J,
                                        unsigned long long budget_pairs, unsigned long long unit_pairs,
                                        const uint32_t* __restrict__ counts, const unsigned long long* __restrict__ gcounts,
                                        uint32_t fold_zero) {
    constexpr uint32_t WAVES = PREDICT_THREADS / 64;
    __shared__ uint32_t above[D1_BINS];        // sample entries in strictly higher bins
    __shared__ uint32_t bitmap[D1_BINS / 32];
    __shared__ uint32_t su[16];
    __shared__ unsigned long long s64[16];
    __shared__ uint32_t sh_gbin, sh_spill, sh_eighth, sh_ns, sh_gap, sh_knext, sh_low;
    __shared__ uint64_t sh_words[D1_BINS / 32 / 64];
    const uint32_t tid = threadIdx.x;
    const uint32_t li = pb.big_layer[big];
    const LayerDesc L = pb.layers[li];

    // this layer's sizes and sample counts are asked for together with the global ones of step (1)
    const uint32_t K = Ktab[(size_t)li * J + min(tid, J - 1u)], K_next = Ktab[(size_t)li * J + min(tid + 1u, J - 1u)];
    uint32_t c[16], csum = 0;
    {
        const uint4* sh4 = reinterpret_cast<const uint4*>(counts + (size_t)big * D1_BINS + tid * 16u);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint4 v = sh4[k];
            c[4 * k] = v.x; c[4 * k + 1] = v.y; c[4 * k + 2] = v.z; c[4 * k + 3] = v.w;
        }
    }
    bool narrow;                                           // the budget is known and at most a 32nd of all entries
    // (1) global threshold bin: the highest bin b with (entries of all layers in bins >= b) >= 1.25 x budget
    // (2.5 x for a wide link, whose sizes the estimate below says little about: most layers spill their eighth there)
    {
        unsigned long long sum = 0;
#pragma unroll
        for (int k = 0; k < 16; ++k) sum += gcounts[tid * 16u + k];
        unsigned long long tot;
        const unsigned long long ex = block_exclusive_scan<unsigned long long>(sum, s64, &tot, WAVES);
        unsigned long long ab = tot - ex - sum;            // entries above this thread's bins
        narrow = budget_pairs != 0ull && budget_pairs <= tot / 32ull;
        const unsigned long long want = narrow ? budget_pairs + budget_pairs / 4ull : budget_pairs * 5ull / 2ull;
        if (tid == 0) { sh_gbin = 0u; sh_knext = 0xFFFFFFFFu; }    // budget beyond everything: bin 0
        __syncthreads();
        if (budget_pairs && ab < want && ab + sum >= want) {
#pragma unroll
            for (int k = 15; k >= 0; --k) {
                const unsigned long long gc = gcounts[tid * 16u + k];      // (one thread's: held by all they would not fit 64 registers)
                if (ab + gc >= want) { sh_gbin = tid * 16u + k; break; }
                ab += gc;
            }
        }
        __syncthreads();
    }
    // (2) this layer's sample: suffix counts
#pragma unroll
    for (int k = 0; k < 16; ++k) csum += c[k];
    uint32_t ns_total;
    const uint32_t cex = block_exclusive_scan<uint32_t>(csum, su, &ns_total, WAVES);
    {
        uint32_t run = cex;
#pragma unroll
        for (int k = 0; k < 16; ++k) { run += c[k]; above[tid * 16u + k] = ns_total - run; }
    }
    if (tid < D1_BINS / 32) bitmap[tid] = 0u;
    __syncthreads();
    const double scale = (double)L.n / (double)(ns_total ? ns_total : 1u);   // population per sample entry
    // Smallest bins with above[bin] < k, i.e. the bins holding the sample entries of ranks k (k >= 1), several at a time: twelve
    // reads of LDS one after another, whatever their number.
    auto find_bins = [&](auto& k, auto& bin) {
        constexpr int N = sizeof(k) / sizeof(k[0]);
#pragma unroll
        for (int q = 0; q < N; ++q) bin[q] = 0u;
#pragma unroll
        for (uint32_t half = D1_BINS / 2u; half; half >>= 1) {
            uint32_t there[N];
#pragma unroll
            for (int q = 0; q < N; ++q) there[q] = above[bin[q] + half - 1u];
#pragma unroll
            for (int q = 0; q < N; ++q) bin[q] += there[q] >= k[q] ? half : 0u;
        }
    };
    // The size the allocation will choose for this layer: an allocation cuts all layers at about
    // the same magnitude, rounded to the grid: the second grid size above this layer's entries in the global bins (the
    // first one left a few of ResNet-50's layers short, which then read g and h again).
    if (narrow && tid < J) {
        const double here = scale * (double)(sh_gbin ? above[sh_gbin - 1u] : ns_total);
        if ((double)K >= here) atomicMin(&sh_knext, K_next);
    }
    __syncthreads();
    if (tid == 0) {
        // Spill down to that size, rounded up to whole cost units (a layer pays for its last unit whole and takes what fits
        // it; one whose entries all lie below the cut still pays for one), plus 3 sigma of the sample count, and to the global
        // threshold bin; at least a four-hundredth of the layer (without a narrow budget the top 2 %) and twice the smallest
        // grid size (plus 3 sigma); at most an eighth of the layer.  What is spilled is written and read again several
        // times: with 2 % of every layer and the entries of 2.5 budgets the Llama-shaped set's k_main took 2412 us and its
        // step 3360, with this 2267 and 3204.  Without the rounding, 66 to 108 of that set's 169 tiled layers ended short with
        // 2 to 6 % of the bytes to spend and read g and h again: steps of 3970 us at 2 % and 5720 at 6 %, now 3460 and 4530.
        const uint32_t K0 = K;
        const double k0s = 2.0 * (double)K0 / scale;
        uint32_t floor_rank = (uint32_t)fmin((double)ns_total, ceil(k0s + 3.0 * sqrt(k0s) + 2.0));
        // (a selection has one target: nothing above it needs a slot)
        floor_rank = max(floor_rank, J == 1u ? 1u : max(1u, ns_total / (narrow ? 400u : 50u)));
        if (narrow) {
            const unsigned long long aim = ((unsigned long long)min(sh_knext, L.n) + unit_pairs - 1ull) / unit_pairs * unit_pairs;
            const double kns = (double)min(aim, (unsigned long long)L.n) / scale;
            floor_rank = max(floor_rank, (uint32_t)fmin((double)ns_total, ceil(kns + 3.0 * sqrt(kns) + 2.0)));
        }
        // never more than the top eighth of the layer: the bin that holds the entry of that rank is spilled only
        // if all of it still lies inside (a layer's candidate region has room for a little more than that share)
        const uint32_t k8 = max(1u, ns_total / 8u);
        const uint32_t rank[3] = {floor_rank, k8, max(1u, above[0])};
        uint32_t bin[3];
        find_bins(rank, bin);
        const uint32_t b = budget_pairs ? min(bin[0], sh_gbin) : bin[0];
        uint32_t bc = bin[1];
        sh_low = bin[2];
        if ((bc == 0u ? ns_total : above[bc - 1u]) > k8) ++bc;     // D1_BINS: nothing is spilled
        sh_spill = max(b, bc);
        sh_eighth = bc;
        // with one target, candidates that cannot serve it are not written: nothing or everything is kept, or more
        // than the eighth that may be spilled
        if (J == 1u && (K0 == 0u || K0 >= L.n || (double)K0 / scale > (double)k8)) sh_spill = D1_BINS;
    }
    __syncthreads();
    uint32_t spill_bin = sh_spill;
    // (3) bins that may hold a candidate's boundary: +-5 sigma of the sample rank, every bin in between.
    // Bin 0 (zeros and the tiniest denormals) never gets a slot here: its squares need the exact
    // accumulators of the full recount.
    if (tid < J) {
        if (K < L.n) {
            const double ks = (double)K / scale;
            const double sg = sqrt(fmax(0.0, ks * (1.0 - ks / (double)ns_total)));
            const double klo = floor(ks - 5.0 * sg) - 2.0, khi = ceil(ks + 5.0 * sg) + 2.0;
            const uint32_t rlo = (uint32_t)fmin((double)ns_total, fmax(1.0, klo));
            const uint32_t rhi = (uint32_t)fmin((double)ns_total, fmax(1.0, khi));
            // (no lower than the smallest entry above bin 0: where many entries are exactly zero, all bins below it are empty)
            const uint32_t rank[2] = {rlo, rhi};
            uint32_t bin[2];
            find_bins(rank, bin);
            const uint32_t btop = bin[0], bbot = max(khi > (double)ns_total ? 0u : bin[1], sh_low);
            // A boundary in the spilled range can also be resolved from the candidates, which is
            // cheap only where few entries lie above it: skip the prediction for the sparse top
            // (fewer than 64 sample entries above), where it would cost many bins.
            const bool sparse_top = ks < 64.0 && bbot >= spill_bin;
            const uint32_t lo = max(bbot, 1u);
            if (!sparse_top && lo <= btop)
                for (uint32_t w = lo >> 5; w <= btop >> 5; ++w)
                    atomicOr(&bitmap[w], (w == lo >> 5 ? ~0u << (lo & 31u) : ~0u) & (w == btop >> 5 ? ~0u >> (31u - (btop & 31u)) : ~0u));
        }
    }
    __syncthreads();
    // (4) slots: runs of consecutive bins from the lowest marked bin (low bins hold the most
    // entries) upward, at most PRE_SLOTS in all.  A run lets the streaming pass find an entry's slot
    // with a subtraction instead of a table look-up.  One run if it reaches the highest marked bin or the spilled range;
    // else two, with the widest stretch of unmarked bins left out between them, and if those still end below both, what
    // is above them is spilled as well, as far as the eighth allows.  (A grid that goes up to nearly all entries, as the
    // paper's, marks 150 bins, with such a stretch at the sparse lower end.  With one run and no more spilled than the
    // budget asks for, every layer was recounted in every round.)
    // What is cut off below the spilled range makes the layer a redo.
    uint8_t* lut = pb.lut1 + (size_t)big * D1_BINS;
    for (uint32_t b = tid; b < D1_BINS; b += 256) lut[b] = (uint8_t)NO_SLOT;
    // lowest and highest marked bin: one bitmap word per thread
    if (tid == 0) { sh_gbin = D1_BINS; sh_ns = 0u; sh_gap = 0u; }      // the first two reused: lowest / highest marked bin
    __syncthreads();
    if (tid < D1_BINS / 32) {
        const uint32_t m = bitmap[tid];
        if (m) {
            atomicMin(&sh_gbin, tid * 32u + (uint32_t)__ffs((int)m) - 1u);
            atomicMax(&sh_ns, tid * 32u + 31u - (uint32_t)__clz((int)m));
        }
    }
    __syncthreads();
    const bool any = sh_gbin < D1_BINS;
    const uint32_t lo_bin = any ? sh_gbin : 0u, hi_bin = sh_ns;
    uint32_t ns = any ? min(PRE_SLOTS, hi_bin - lo_bin + 1u) : 0u, run_a = ns, lo_b = 0u;
    if (any && lo_bin + PRE_SLOTS <= min(hi_bin, spill_bin - 1u)) {    // (the same in every thread; spill_bin is never 0 then)
        // the widest stretch that ends before a marked bin: its width, then that bin
        const uint32_t m = tid < D1_BINS / 32 ? bitmap[tid] : 0u;
        const uint64_t words = ballot(m != 0u);
        if (tid < D1_BINS / 32 && lane_id() == 0u) sh_words[tid >> 6] = words;
        __syncthreads();
        if (m) {
            // bins whose neighbour below is not marked
            uint32_t starts = m & ~((m << 1) | (tid ? bitmap[tid - 1u] >> 31 : 0u)), widest = 0u;
            for (; starts; starts &= starts - 1u) {
                const uint32_t at = (uint32_t)__ffs((int)starts) - 1u, low = m & ((1u << at) - 1u), b = tid * 32u + at;
                uint32_t w = tid, word = low;
                if (!low) {
                    // the marked word before this one
                    const uint64_t here = sh_words[tid >> 6] & ((1ull << lane_id()) - 1ull);
                    const bool one = here != 0ull || (tid >= 64u && sh_words[0] != 0ull);
                    if (!one) continue;                                // (the lowest marked bin)
                    w = here ? (tid & ~63u) + 63u - (uint32_t)__clzll((long long)here) : 63u - (uint32_t)__clzll((long long)sh_words[0]);
                    word = bitmap[w];
                }
                const uint32_t before = w * 32u + 31u - (uint32_t)__clz((int)word);
                widest = max(widest, ((b - before - 1u) << D1_BITS) | b);
            }
            atomicMax(&sh_gap, widest);
        }
        __syncthreads();
        const uint32_t gap = sh_gap >> D1_BITS;
        uint32_t end = lo_bin + PRE_SLOTS;                             // first bin above the runs
        if (gap) {
            const uint32_t first_b = sh_gap & (D1_BINS - 1u);
            if (first_b - gap - lo_bin < PRE_SLOTS) {
                lo_b = first_b;
                run_a = lo_b - gap - lo_bin;
                ns = min(PRE_SLOTS, run_a + (hi_bin - lo_b + 1u));
                end = lo_b + (ns - run_a);
            }
        }
        if (end <= min(hi_bin, spill_bin - 1u)) spill_bin = min(spill_bin, max(end, sh_eighth));
    }
    if (tid < ns) {
        const uint32_t b = tid < run_a ? lo_bin + tid : lo_b + (tid - run_a);
        lut[b] = (uint8_t)tid;
        pb.slot_bin[(size_t)big * SLOT_STRIDE + tid] = b;
    }
    if (tid == 0) {
        LayerState st;
        st.spill_bin = spill_bin; st.nslots_d = ns; st.nslots_t = 0; st.redo = 0;
        st.spill_cnt = 0; st.spill_valid = 0; st.slot_lo = lo_bin | (lo_b << 16); st.run_a = run_a;
        pb.state[big] = st;
    }
    if (fold_zero) {
        // chunk records start out as "nothing spilled": every workgroup clears an equal share of all layers' records
        // (a layer's own workgroup clearing them made the largest layer's the last to finish by far)
        const uint32_t per = (pb.nchunks_total + nbig - 1u) / nbig;
        const uint32_t c_lo = big * per, c_hi = min(pb.nchunks_total, c_lo + per);
        for (uint32_t c = c_lo + tid; c < c_hi; c += 256) pb.rec_cnt[c] = 0u;
        if (tid == 0) { pb.layer_flag[big] = 0u; pb.cursor[big] = 0u; pb.spill_over[big] = 0u; pb.tiles_done[big] = 0u; }
        if (big == 0u && tid < 4u) pb.diag[tid] = 0u;
        if (big == 0u && tid == 4u) *pb.fresh = 0u;
    }
}

// One launch for both: a workgroup per tiled layer that predicts, and, from `nbig` on, one per small layer that profiles it
// (without an err_table there are none of these).  The predictions are a few dozen workgroups that wait for memory; on a
// stream of their own beside the kernels behind the pass the small layers cost the two events, 6 us each, that bring them
// there and back.  (GPT-2-shaped, 98 small layers: predictions 14 us, small layers 15, both 17; since the sort takes one instruction a
// value and step and the searches run side by side, the predictions are through after 10, the small layers after 13, ResNet-18's after 21.)
// (at least eight waves a SIMD: two workgroups to a compute unit)
__global__ __launch_bounds__(SMALL_THREADS, 8) void k_predict(ProfileBuffers pb, uint32_t nbig, const uint32_t* Ktab, uint32_t J,
                                                           unsigned long long budget_pairs, unsigned long long unit_pairs,
                                                           const uint32_t* __restrict__ counts,
                                                           const unsigned long long* __restrict__ gcounts, uint32_t fold_zero,
                                                           double* err_table) {
    if (blockIdx.x >= nbig) small_profile(pb, blockIdx.x - nbig, Ktab, J, err_table);
    else if (threadIdx.x < PREDICT_THREADS) predict(pb, blockIdx.x, nbig, Ktab, J, budget_pairs, unit_pairs, counts, gcounts, fold_zero);
}

// ---------------------------------------------------------------------------------------------
// The streaming pass.  Persistent grid: workgroup w owns a contiguous range of chunks (shares.h), walks it
// layer by layer, and keeps that layer's histograms in LDS as one array of packed entries
// [count:20 | sum:44] of (significand^2 >> 24): 4096 digit-1 bins, then up to PRE_SLOTS slots x 128 digit-2
// bins.  Entries whose bin has a slot are counted only there.  Bin 0 (zeros, tiniest denormals)
// keeps exact squares in a separate accumulator.  One wave handles one chunk at a time: 4 quads per
// lane, one LDS atomic per entry, then spilling, ranked by prefix scans over the lanes, of the entries at or above the layer's
// spill bin, staged through LDS so that the candidate writes are coalesced.
//
// The packed sums drop the low 24 bits of each square: the true sum of (square >> 16) lies in
// [256 S, 256 S + 256 count); k_reduce_parts stores the midpoint and the scans widen their bounds by
// half that interval (2^-23 relative).
constexpr uint32_t PK_ENTRIES = D1_BINS + PRE_SLOTS * D2_BINS;     // 17920 entries, 140 KB
constexpr uint32_t STAGE = 128;                                    // candidates a wave's window holds
constexpr uint32_t PART_STRIDE = PK_ENTRIES + 8;                   // entries of one part: the LDS array, then the bin-0 sum

// A part's head: whether there is one, then a bit per block of PART_BLOCK entries: whether it was written with 64 bits an
// entry (a digit-1 block without the bit has no entry, a slot's without it is packed).
constexpr uint32_t PART_BLOCK = 128;
constexpr uint32_t PART_HEAD = 8;
static_assert(PART_BLOCK == D2_BINS && D1_BINS % PART_BLOCK == 0 && (PK_ENTRIES / PART_BLOCK + 31) / 32 < PART_HEAD, "a slot is a block");

// digit-1 bin of a slot of the two runs
__device__ __forceinline__ uint32_t slot_bin_of(const LayerState& st, uint32_t s) {
    return s < st.run_a ? (st.slot_lo & 0xFFFFu) + s : (st.slot_lo >> 16) + (s - st.run_a);
}
// An entry of a slot in 32 bits, [count:10 | sum:22]: every significand of the entry is M 2^12 + d with the same M, d < 2^12, so
// (its square >> 24) is M^2 and less than 2^13 more; the sum of what is more.  False where the count or that sum is too
// large, and for the exponents 0 and 255, whose terms are others.
constexpr uint32_t NARROW_SHIFT = 22;
__device__ __forceinline__ uint32_t slot_square(uint32_t bin, uint32_t d2) {
    const uint32_t m = 0x800u | ((bin & 15u) << D2_BITS) | d2;
    return m * m;
}
__device__ __forceinline__ bool pack_slot_entry(uint32_t bin, uint32_t d2, unsigned long long e, uint32_t& packed) {
    const uint32_t cnt = (uint32_t)(e >> 44), exponent = bin >> 4;
    const unsigned long long more = (e & PK_MASK) - (unsigned long long)cnt * slot_square(bin, d2);
    packed = (cnt << NARROW_SHIFT) | (uint32_t)more;
    return cnt < (1u << (32u - NARROW_SHIFT)) && more < (1ull << NARROW_SHIFT) && exponent != 0u && exponent != 255u;
}

__device__ __forceinline__ unsigned long long pk_term(uint32_t key) {
    const uint32_t m = key & 0x7FFFFFu, e = key >> 23;
    const uint32_t m24 = e ? (m | 0x800000u) : m;
    return e == 255u ? (unsigned long long)(m != 0u) : ((unsigned long long)m24 * m24) >> PK_SHIFT;
}

struct MainCtx {
    unsigned long long* pk;
    unsigned long long* sq0;
    // a run of slot bins: 19-bit key prefix of its first digit-2 entry, and how many digit-2 entries it has: a key is in
    // one of its bins iff (key >> 12) - lo19 < span
    uint32_t lo19, span;   // the first run: LDS entries D1_BINS..
    uint32_t lo19b, spanb; // the second run, right behind it (spanb = 0: there is none)
    uint32_t spill_key;
};

// LDS entry of a key: inside a run of slot bins the digit-2 entries of consecutive bins are
// consecutive 19-bit prefixes, so the entry is the prefix minus the run's first one
template <bool TWO>
__device__ __forceinline__ uint32_t main_entry(const MainCtx& cx, uint32_t k) {
    const uint32_t rel = (k >> D2_SHIFT) - cx.lo19;
    const uint32_t e = rel < cx.span ? D1_BINS + rel : (k >> D1_SHIFT);
    if (!TWO) return e;
    const uint32_t relb = (k >> D2_SHIFT) - cx.lo19b;
    return relb < cx.spanb ? D1_BINS + cx.span + relb : e;
}

// the same for all entries of a chunk that lies inside the layer and holds only normal numbers
template <bool TWO>
__device__ __forceinline__ void main_count_plain(const MainCtx& cx, const float (&x)[NQ][4], uint32_t (&selm)[NQ]) {
#pragma unroll
    for (int u = 0; u < (int)NQ; ++u) {
        uint32_t sel = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t k = key_of(x[u][c]);
            const uint32_t m24 = (k & 0x7FFFFFu) | 0x800000u;
            // the shifted square has 24 bits: as a 32-bit value it is the low word of the packed
            // operand and the count's 1 is a constant high word
            const unsigned long long sq = (unsigned long long)m24 * m24;
            const uint32_t t = __builtin_amdgcn_alignbit((uint32_t)(sq >> 32), (uint32_t)sq, PK_SHIFT);
            atomicAdd(&cx.pk[main_entry<TWO>(cx, k)], PK_ONE | (unsigned long long)t);
            sel |= (k >= cx.spill_key ? 1u : 0u) << c;
        }
        selm[u] = sel;
    }
}

// histogram updates and spill flags of one chunk.  A chunk that lies inside the layer and holds
// only normal numbers (no zeros, denormals, Inf, NaN) takes a branch-free path.
template <bool TWO>
__device__ __forceinline__ void main_count(const MainCtx& cx, const float (&x)[NQ][4], uint32_t valid,
                                           uint32_t (&selm)[NQ]) {
    // exponent field 0 or 255 anywhere in the lane's 16 keys: smallest and largest key
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
    for (int u = 0; u < (int)NQ; ++u) {
        const uint32_t k0 = key_of(x[u][0]), k1 = key_of(x[u][1]), k2 = key_of(x[u][2]), k3 = key_of(x[u][3]);
        kmin = min(min(kmin, k0), min(min(k1, k2), k3));
        kmax = max(max(kmax, k0), max(max(k1, k2), k3));
    }
    const bool special = kmin < 0x00800000u || kmax >= 0x7F800000u;
    const bool plain = ballot(special || valid != (1u << (4 * NQ)) - 1u) == 0;
    if (plain) {
        main_count_plain<TWO>(cx, x, selm);
        return;
    }
#pragma unroll
    for (int u = 0; u < (int)NQ; ++u) {
        selm[u] = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (!(valid & (1u << (4 * u + c)))) continue;
            const uint32_t k = key_of(x[u][c]);
            if ((k >> D1_SHIFT) != 0u) {
                atomicAdd(&cx.pk[main_entry<TWO>(cx, k)], PK_ONE | pk_term(k));
            } else {
                atomicAdd(&cx.pk[0], PK_ONE);
                if (k) atomicAdd(cx.sq0, sq_exact(k));
            }
            if (k >= cx.spill_key) selm[u] |= 1u << c;
        }
    }
}

// Spilling.  Stores cost this pass several times their bytes (1.2 % of the entries: 330 us of 1980 on 10 GB of g and h; a plain
// read of the same bytes takes 1470), most of all stores of partial lines, which are written back and fetched again among
// the streaming reads.  And a store in the loop makes every wait for the next chunk's loads a wait for its acknowledgement
// as well, and a returning global atomic per reservation serialises thousands of waves on one address.  So:
//   * the workgroup owns the slice of the layer's candidate region that corresponds to its chunks,
//     handed out in units of a 128-byte line (spill_slice in segment.h, also for short slices); a slice that runs
//     out marks the layer's spill as incomplete (spill_over) and the layer is served by the passes
//     that read g and h instead, like any other misprediction;
//   * a candidate is six bytes: x, and its place in the chunk; a wave takes blocks from an LDS cursor, collects candidates
//     in an LDS window and writes 64 of them, whole lines, as soon as they are there (a chunk with more than 64 entries
//     takes exactly the units it needs and writes them at once);
//   * chunk records wait in LDS.  A chunk's candidates are always contiguous.
// (10 GB of g and h, 1.1 and 9 % of the entries: eight bytes each in runs of whatever a window of 128 held 2040 and 2770 us;
// six bytes and whole lines 1906 and 2593, nontemporal 1807 and 2193; pairs of index and x, nontemporal, 1840 and 2210, but
// the kernels that look at x alone read twice as much then.  1 GB, 1.1 %: 186, 181 and 185.  Nothing written: 1660 and 172.)
constexpr uint32_t PEND = 16;                   // chunk records a wave holds back

struct WaveSpill {
    float* win_x;         // LDS window: the block's entries from `flushed` on, entry e at e % STAGE
    uint16_t* win_i;
    uint32_t* pend;       // LDS: PEND x (chunk, start, count)
    uint32_t* lds_cursor; // units handed out in this workgroup's slice
    uint32_t* over;       // the layer's spill_over flag
    SpillSlice slice;     // (chunk records are relative to the layer's region like the slice's first entry)
    uint32_t blk;         // region-relative start of the current block (valid if have_blk)
    uint32_t fill;        // entries in the block
    uint32_t flushed;     // of which already written: all below the last multiple of SPILL_RUN
    uint32_t npend;
    bool have_blk;
};

template <bool STREAM>
__device__ __forceinline__ void store_candidate(const ProfileBuffers& pb, uint64_t o, float x, uint16_t i) {
    if (STREAM) {
        __builtin_nontemporal_store(x, pb.tmp_x + o);
        __builtin_nontemporal_store(i, pb.tmp_i + o);
    } else {
        pb.tmp_x[o] = x;
        pb.tmp_i[o] = i;
    }
}

// the block's entries up to `upto` (at most SPILL_RUN of them)
template <bool STREAM>
__device__ __forceinline__ void spill_write(const ProfileBuffers& pb, WaveSpill& ws, uint64_t tmp0, uint32_t upto) {
    wave_sync_lds();
    const uint32_t k = ws.flushed + lane_id();
    if (k < upto) store_candidate<STREAM>(pb, tmp0 + ws.blk + k, ws.win_x[k % STAGE], ws.win_i[k % STAGE]);
    ws.flushed = upto;
    wave_sync_lds();
}
__device__ __forceinline__ void spill_records(const ProfileBuffers& pb, WaveSpill& ws) {
    wave_sync_lds();
    if (lane_id() < ws.npend) {
        const uint32_t* r = ws.pend + 3u * lane_id();
        pb.rec_start[r[0]] = r[1];
        pb.rec_cnt[r[0]] = r[2];
    }
    ws.npend = 0;
    wave_sync_lds();
}

// take room for `entries` consecutive entries of the slice; returns the region-relative index of the
// first.  *ok is false when the slice has no room left for them: nothing may be written then, and the
// layer is marked.
__device__ __forceinline__ uint32_t spill_take(WaveSpill& ws, uint32_t entries, bool* ok) {
    const uint32_t nu = (entries + (1u << ws.slice.unit_log) - 1u) >> ws.slice.unit_log;
    uint32_t b = 0;
    if (lane_id() == 0) b = atomicAdd(ws.lds_cursor, nu);
    b = __builtin_amdgcn_readfirstlane(b);
    *ok = b + nu <= ws.slice.units;             // (the cursor grows by at most 128 units per chunk: no wrap)
    if (!*ok && lane_id() == 0) *ws.over = 1u;
    return ws.slice.first + (b << ws.slice.unit_log);
}

// One chunk of the streaming pass for one wave: histogram updates, ranks of the entries to spill,
// space for them, window writes, chunk record.
template <bool TWO, bool STREAM>
__device__ __forceinline__ void main_chunk(const ProfileBuffers& pb, const MainCtx& cx, const LayerDesc& L, WaveSpill& ws,
                                           uint32_t chunk, const float (&x)[NQ][4], uint32_t valid) {
    const uint32_t lane = lane_id();
    uint32_t selm[NQ];
    main_count<TWO>(cx, x, valid, selm);
    // ranks in index order (quad, lane, element): per quad a prefix sum over the lanes of the lane's
    // count (0..4); two quads share a scan in 16-bit fields (a quad holds at most 256)
    static_assert(NQ == 4, "two packed scans cover four quads");
    const uint32_t n0 = __popc(selm[0]), n1 = __popc(selm[1]), n2 = __popc(selm[2]), n3 = __popc(selm[3]);
    const uint32_t s01 = wave_scan_add_u32(n0 | (n1 << 16)), s23 = wave_scan_add_u32(n2 | (n3 << 16));
    const uint32_t t01 = (uint32_t)__builtin_amdgcn_readlane((int)s01, 63), t23 = (uint32_t)__builtin_amdgcn_readlane((int)s23, 63);
    const uint32_t t0 = t01 & 0xFFFFu, t1 = t01 >> 16, t2 = t23 & 0xFFFFu;
    const uint32_t total = t0 + t1 + t2 + (t23 >> 16);
    uint32_t rowbase[NQ];
    rowbase[0] = (s01 & 0xFFFFu) - n0;
    rowbase[1] = t0 + (s01 >> 16) - n1;
    rowbase[2] = t0 + t1 + (s23 & 0xFFFFu) - n2;
    rowbase[3] = t0 + t1 + t2 + (s23 >> 16) - n3;
    if (total == 0) return;                      // records start out as "nothing spilled"
    if (total <= SPILL_RUN) {
        if (ws.npend == PEND) spill_records(pb, ws);
        if (!ws.have_blk || ws.fill + total > ws.slice.block) {
            if (ws.have_blk) spill_write<STREAM>(pb, ws, L.tmp0, ws.fill);
            bool ok;
            ws.blk = spill_take(ws, ws.slice.block, &ok);
            ws.fill = 0; ws.flushed = 0; ws.have_blk = ok;
            if (!ok) return;                     // the chunk's record stays "nothing spilled"; the layer is marked
        }
        const uint32_t at = ws.fill;
        // Few entries are spilled, so a lane rarely holds more than one per quad: write in rounds,
        // every lane its next selected entry of the quad (ascending element), until no lane has one
        // left.  On average that is fewer than two wave-wide writes per quad instead of four.
#pragma unroll
        for (int u = 0; u < (int)NQ; ++u) {
            uint32_t m = selm[u];
            uint32_t pos = at + rowbase[u];
            const uint32_t place = u * 256u + lane * 4u;
            while (ballot(m != 0u)) {
                if (m) {
                    const float xv = (m & 1u) ? x[u][0] : (m & 2u) ? x[u][1] : (m & 4u) ? x[u][2] : x[u][3];
                    ws.win_x[pos % STAGE] = xv;
                    ws.win_i[pos % STAGE] = (uint16_t)(place + (uint32_t)__builtin_ctz(m));
                    ++pos;
                    m &= m - 1u;
                }
            }
        }
        if (lane == 0) {
            ws.pend[3 * ws.npend] = chunk;
            ws.pend[3 * ws.npend + 1] = ws.blk + at;
            ws.pend[3 * ws.npend + 2] = total;
        }
        ws.fill += total;
        ws.npend += 1;
        // (fewer than SPILL_RUN entries were waiting, so the window holds them all and one run is written at most)
        const uint32_t run = ws.flushed / SPILL_RUN * SPILL_RUN + SPILL_RUN;
        if (ws.fill >= run) spill_write<STREAM>(pb, ws, L.tmp0, run);
    } else {
        // a dense chunk: units of its own, written through the window in rounds; the block goes on afterwards
        if (ws.have_blk) spill_write<STREAM>(pb, ws, L.tmp0, ws.fill);
        bool ok;
        const uint32_t start = spill_take(ws, total, &ok);
        if (!ok) return;
        const uint64_t base = L.tmp0 + start;
        for (uint32_t r0 = 0; r0 < total; r0 += STAGE) {
#pragma unroll
            for (int u = 0; u < (int)NQ; ++u) {
                uint32_t pos = rowbase[u];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (selm[u] & (1u << c)) {
                        const uint32_t k = pos - r0;
                        if (k < STAGE) {
                            ws.win_x[k] = x[u][c];
                            ws.win_i[k] = (uint16_t)(u * 256u + lane * 4u + c);
                        }
                        ++pos;
                    }
                }
            }
            wave_sync_lds();
#pragma unroll
            for (uint32_t k = lane; k < STAGE; k += 64) {
                if (r0 + k < total) store_candidate<STREAM>(pb, base + r0 + k, ws.win_x[k], ws.win_i[k]);
            }
            wave_sync_lds();
        }
        if (lane == 0) { pb.rec_start[chunk] = start; pb.rec_cnt[chunk] = total; }
    }
}

// How far a workgroup may go with one histogram: segment.h.
struct Segment {
    uint32_t end;          // end of the workgroup's share of the layer
    uint32_t used;         // entries of the histogram
    uint32_t* next_chunk;  // LDS: first chunk no wave has taken yet
    uint32_t* allowed;     // LDS: chunks below it may be counted
    uint32_t* state;       // LDS: LIMIT_*
};
__device__ __forceinline__ uint32_t lds_load(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }

// A wave's view of a stretch's limit (stretch_limit): every value is the same in all its lanes.
struct StretchWave {
    const MainCtx& cx;
    const Segment& sg;
    static constexpr uint32_t OPEN = 2u * FUSED_WAVES;
    __device__ __forceinline__ uint32_t state() const { return __builtin_amdgcn_readfirstlane(lds_load(sg.state)); }
    __device__ __forceinline__ uint32_t allowed() const { return __builtin_amdgcn_readfirstlane(lds_load(sg.allowed)); }
    // What is not in the counts that most() reads: chunks from taken() on, and of those before it the one that a wave is at and
    // the one it has taken ahead (a wave's LDS instructions run in order: when it takes a chunk, all but its last are counted).
    __device__ __forceinline__ uint32_t taken() const {
        const uint32_t t = __builtin_amdgcn_readfirstlane(lds_load(sg.next_chunk));
        wave_sync_lds();
        return t;
    }
    __device__ __forceinline__ uint32_t most() const {
        uint32_t m = 0;
        for (uint32_t b = lane_id(); b < sg.used; b += 64) m = max(m, lds_load(reinterpret_cast<const uint32_t*>(cx.pk) + 2 * b + 1) >> 12);
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) m = max(m, (uint32_t)__shfl_xor(m, d, 64));
        return __builtin_amdgcn_readfirstlane(m);
    }
    __device__ __forceinline__ bool claim() const {
        uint32_t was = 0;
        if (lane_id() == 0) was = atomicCAS(sg.state, (uint32_t)LIMIT_FREE, (uint32_t)LIMIT_READING);
        return __builtin_amdgcn_readfirstlane(was) == LIMIT_FREE;
    }
    __device__ __forceinline__ void allow(uint32_t end) const {
        if (lane_id() == 0) __hip_atomic_store(sg.allowed, end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ void release(uint32_t next) const {
        if (lane_id() == 0) __hip_atomic_store(sg.state, next, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        wave_sync_lds();
    }
    __device__ __forceinline__ void pause() const { __builtin_amdgcn_s_sleep(1); }
};

// A wave's chunks of a segment: its first one, then what the segment's counter hands out.  Returns where the segment ends as
// far as the wave knows: sg.end, or where the stretch does.
template <bool TWO, bool STREAM>
__device__ __forceinline__ uint32_t main_walk(const ProfileBuffers& pb, const MainCtx& cx, const LayerDesc& L, WaveSpill& ws,
                                              uint32_t chunk, const Segment& sg) {
    uint32_t limit = __builtin_amdgcn_readfirstlane(lds_load(sg.allowed));
    for (;;) {
        if (limit < sg.end && chunk + LIMIT_NEAR >= limit) {
            StretchWave w{cx, sg};
            limit = stretch_limit(w, chunk, limit, sg.end, StretchWave::OPEN);
        }
        if (chunk >= limit) return limit;
        uint32_t taken = 0;
        if (lane_id() == 0) taken = atomicAdd(sg.next_chunk, 1u);
        QuadGH q[NQ];
        float x[NQ][4];
        uint32_t valid = 0;
        load_chunk<NQ>(L, (chunk - L.chunk0) * CHUNK, q, valid);
#pragma unroll
        for (int u = 0; u < (int)NQ; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) x[u][c] = q[u].g[c] - q[u].h[c];
        main_chunk<TWO, STREAM>(pb, cx, L, ws, chunk, x, valid);
        chunk = __builtin_amdgcn_readfirstlane(taken);
    }
}

// STREAM: the candidates are stored nontemporally.
template <bool STREAM>
__global__ __launch_bounds__(FUSED_THREADS) void k_main(ProfileBuffers pb) {
    __shared__ __align__(16) unsigned long long pk[PK_ENTRIES];   // 140 KB
    __shared__ unsigned long long sq0;
    __shared__ float stage_x[FUSED_WAVES * STAGE];                // 8 KB and 4 KB: per-wave block windows
    __shared__ uint16_t stage_i[FUSED_WAVES * STAGE];
    __shared__ uint32_t pend[FUSED_WAVES * PEND * 3];             // 3 KB
    __shared__ uint32_t lds_cursor;
    __shared__ uint32_t next_chunk, allowed, limit_state;         // Segment
    __shared__ uint32_t head[PART_HEAD];
    const uint32_t tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const MainShare share = pb.shares[blockIdx.x];
    const uint32_t c_end = pb.shares[blockIdx.x + 1u].chunk;
    uint32_t cur = share.chunk, part = share.part0, li = share.li;
    for (uint32_t big = share.big, next_li; cur < c_end; ++big, li = next_li) {
        next_li = pb.big_layer[big + 1u];
        const LayerDesc L = pb.layers[li];
        const LayerState st = pb.state[big];
        const uint32_t seg_end = min(c_end, L.chunk0 + L.nchunks);
        const uint32_t used = D1_BINS + st.nslots_d * D2_BINS;
        const Segment sg{seg_end, used, &next_chunk, &allowed, &limit_state};
        if (tid == 0) lds_cursor = 0u;
        MainCtx cx;
        cx.pk = pk; cx.sq0 = &sq0;
        cx.lo19 = (st.slot_lo & 0xFFFFu) << (D1_SHIFT - D2_SHIFT); cx.span = st.run_a * D2_BINS;
        cx.lo19b = (st.slot_lo >> 16) << (D1_SHIFT - D2_SHIFT); cx.spanb = (st.nslots_d - st.run_a) * D2_BINS;
        cx.spill_key = st.spill_bin >= D1_BINS ? 0x80000000u : (st.spill_bin << D1_SHIFT);
        WaveSpill ws;
        ws.win_x = stage_x + wave * STAGE; ws.win_i = stage_i + wave * STAGE;
        ws.pend = pend + wave * PEND * 3; ws.lds_cursor = &lds_cursor;
        ws.over = pb.spill_over + big;
        ws.slice = spill_slice(L.tmp0, cur - L.chunk0, seg_end - cur);
        ws.blk = 0; ws.fill = 0; ws.flushed = 0; ws.npend = 0; ws.have_blk = false;

        // (Fetching the wave's next chunk while the current one is worked on was tried at 16, 12 and 8
        // waves per workgroup: no gain.)
        // Waves take chunks from a counter, not in a fixed rotation: a wave's pace varies with what it
        // finds (spills, flushes, memory), and with fixed shares the segment's end waited for its slowest
        // wave for a good tenth of the pass.  The next chunk is asked for before the current one is
        // worked on, so the counter's round trip is never waited for.  No result depends on which wave
        // had which chunk.
        // (one copy of the loop per number of slot runs: testing for the second run in the loop cost 2 % of the pass)
        uint32_t made = 0;                          // parts of this segment
        for (uint32_t start = cur; start < seg_end;) {
            for (uint32_t b = tid; b < used; b += FUSED_THREADS) pk[b] = 0ull;
            if (tid == 0) { sq0 = 0ull; next_chunk = start + FUSED_WAVES; allowed = min(seg_end, start + PK_MAX_CHUNKS); limit_state = LIMIT_FREE; }
            if (tid < PART_HEAD) head[tid] = tid ? 0u : 1u;
            __syncthreads();
            uint32_t stop;
            if (cx.spanb == 0u) stop = main_walk<false, STREAM>(pb, cx, L, ws, start + wave, sg);
            else stop = main_walk<true, STREAM>(pb, cx, L, ws, start + wave, sg);
            if (stop == seg_end) {
                if (ws.have_blk) spill_write<STREAM>(pb, ws, L.tmp0, ws.fill);
                spill_records(pb, ws);
            }
            __syncthreads();
            // The histogram goes out as one "part" of the layer; k_reduce_parts adds the parts up.  (Adding into the layer's
            // arrays with global atomics from here held every workgroup of a layer up on the same cache lines at the same
            // moment.)  A wave takes 128 entries at a time.  Of the digit-1 bins, blocks without an entry stay out.  An entry of
            // a slot is packed into 32 bits where its block allows it: all its squares share their top 12 bits, so their sum is
            // known from the count but for 22 bits.  (146 KB a part whatever is in it made 45 MB of stores at the pass's end, when
            // nothing is left to hide them behind.)
            // Stores that go through to memory at once: left dirty in the L2, the lines were written back one by one among the
            // streaming reads (10 GB of g and h without candidates, 1512 parts: 1735 us with ordinary stores, 1640 so, 1660
            // nontemporal, 1510 without any).
            {
                typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                constexpr int SC1 = 16;                                              // device scope
                __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(pb.parts + (size_t)(part + made) * PART_STRIDE, 0, PART_STRIDE * 8u, 0x00027000);
                const uint32_t lane = lane_id(), blocks = used / PART_BLOCK;
                const ulonglong2* pk2 = reinterpret_cast<const ulonglong2*>(pk);
                for (uint32_t k = wave; k < blocks; k += FUSED_WAVES) {
                    const ulonglong2 e = pk2[k * (PART_BLOCK / 2u) + lane];
                    const int at = (int)(k * PART_BLOCK * 8u);
                    bool narrow = false;
                    if (k >= D1_BINS / PART_BLOCK) {
                        const uint32_t s = k - D1_BINS / PART_BLOCK, bin = slot_bin_of(st, s);
                        uint32_t n0, n1;
                        const bool ok = pack_slot_entry(bin, 2u * lane, e.x, n0) && pack_slot_entry(bin, 2u * lane + 1u, e.y, n1);
                        narrow = ballot(!ok) == 0ull;
                        if (narrow) {
                            u32x2 v;
                            v.x = n0; v.y = n1;
                            __builtin_amdgcn_raw_buffer_store_b64(v, out, at + (int)(lane * 8u), 0, SC1);
                        }
                    } else if (ballot((e.x | e.y) != 0ull) == 0ull) {
                        continue;
                    }
                    if (!narrow) {
                        u32x4 v;
                        v.x = (uint32_t)e.x; v.y = (uint32_t)(e.x >> 32); v.z = (uint32_t)e.y; v.w = (uint32_t)(e.y >> 32);
                        __builtin_amdgcn_raw_buffer_store_b128(v, out, at + (int)(lane * 16u), 0, SC1);
                        if (lane == 0) atomicOr(&head[1u + k / 32u], 1u << (k % 32u));
                    }
                }
                if (tid == 0) pb.parts[(size_t)(part + made) * PART_STRIDE + PK_ENTRIES] = sq0;
            }
            ++made;
            // the next stretch clears the LDS array: its reads above must be done, the stores need not be
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (tid < PART_HEAD) pb.part_head[(size_t)(part + made - 1u) * PART_HEAD + tid] = head[tid];
            start = stop;
        }
        // there is room for a part every PK_MAX_CHUNKS chunks: those that are not there
        const uint32_t planned = (seg_end - cur + PK_MAX_CHUNKS - 1u) / PK_MAX_CHUNKS;
        for (uint32_t k = made + tid; k < planned; k += FUSED_THREADS) pb.part_head[(size_t)(part + k) * PART_HEAD] = 0u;
        part += planned;
        cur = seg_end;
    }
}

// ---------------------------------------------------------------------------------------------
// Sum of a layer's parts, written in the layout the scans read: digit-1 counts and sums, then the
// digit-2 tables of all SLOT_STRIDE slots (zero beyond the slots the pass counted, where k_hist2c
// adds).  Counts as they are; sums as midpoints in units of 2^16 (exponent 255: the NaN count;
// bin 0: the exact squares).
// Most layers have a handful of parts, and what a block takes is a chain of memory round trips (the layer's state and the
// parts' heads, the parts, the stores): a wave looks after a block by itself.  A layer of more than REDUCE_WAVE_PARTS parts
// has a workgroup to every block, whose waves take a quarter of the parts each.  The host lists these layers first (reduce_layers).
// (us with a workgroup to every block of every layer, and now: ResNet-50 14.6 and 10.5, GPT-2-shaped, whose embedding has 80
// parts, 14.2 and 12.9, Llama-shaped 38 and 25.  The line, us by events with waves up to 8, 16 and 32 parts: Llama-shaped 35.0, 25.6,
// 25.8, ResNet-50 12.6, 12.6, 14.0, with a wide link 14.2, 14.4, 16.4, ResNet-18 with 50 ratios 14.4, 14.1, 14.7.  With a list of the
// workgroups in the place of one of the layers, Llama-shaped 27.5, ResNet-50 13.0.)
constexpr uint32_t LAYER_ENTRIES = D1_BINS + SLOT_STRIDE * D2_BINS;
constexpr uint32_t REDUCE_ENTRIES = 128;        // entries of a block: two per lane
constexpr uint32_t REDUCE_BLOCKS = LAYER_ENTRIES / REDUCE_ENTRIES, REDUCE_WAVE_PARTS = 16;
inline uint32_t reduce_workgroups(uint32_t nbig, uint32_t nsplit) { return nsplit * REDUCE_BLOCKS + (nbig - nsplit) * (REDUCE_BLOCKS / 4u); }
static_assert(REDUCE_BLOCKS * REDUCE_ENTRIES == LAYER_ENTRIES && REDUCE_BLOCKS % 4u == 0u, "four whole blocks to a workgroup");

// Counts and sums of lanes' two entries e, e + 1 as the scans read them.
__device__ __forceinline__ void reduce_store(const ProfileBuffers& pb, uint32_t big, uint32_t blk, uint32_t lane, const unsigned long long (&cnt)[2],
                                             const unsigned long long (&t)[2], unsigned long long zeros_sq) {
    const uint32_t e = blk * REDUCE_ENTRIES + 2u * lane;
    const uint32_t slot_bin = blk < D1_BINS / REDUCE_ENTRIES ? 0u : pb.slot_bin[(size_t)big * SLOT_STRIDE + (blk - D1_BINS / REDUCE_ENTRIES)];
    unsigned long long slot_sq = 0;               // this lane's share of the slot's total (blocks beyond the digit-1 bins)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const uint32_t eu = e + (uint32_t)u;
        unsigned long long s2 = 0;
        if (cnt[u]) {
            const uint32_t bin = eu < D1_BINS ? eu : slot_bin;
            if ((bin >> 4) == 255u) {
                s2 = t[u];
            } else if (eu == 0u) {
                s2 = zeros_sq;
            } else {
                s2 = (t[u] << 8) + (cnt[u] << 7);
            }
        }
        if (eu < D1_BINS) {
            pb.cnt1[(size_t)big * D1_BINS + eu] = (uint32_t)cnt[u];
            reinterpret_cast<unsigned long long*>(pb.sq1)[(size_t)big * D1_BINS + eu] = s2;
        } else {
            const size_t o = (size_t)big * SLOT_STRIDE * D2_BINS + (eu - D1_BINS);
            pb.cnt2[o] = (uint32_t)cnt[u];
            reinterpret_cast<unsigned long long*>(pb.sq2)[o] = s2;
            slot_sq += s2;
        }
    }
    // a block beyond the digit-1 bins holds exactly one slot: its totals, which stand for the slot's bin in the
    // digit-1 histogram (the pass counts an entry of a slot bin in the slot only), go out with it
    static_assert(REDUCE_ENTRIES == D2_BINS && D1_BINS % REDUCE_ENTRIES == 0, "one block per slot");
    if (blk >= D1_BINS / REDUCE_ENTRIES) {
        unsigned long long slot_cnt = cnt[0] + cnt[1];
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            slot_cnt += __shfl_xor(slot_cnt, d, 64);
            slot_sq += __shfl_xor(slot_sq, d, 64);
        }
        if (lane == 0) {
            const size_t o = (size_t)big * SLOT_STRIDE + (blk - D1_BINS / REDUCE_ENTRIES);
            pb.slot_cnt[o] = (uint32_t)slot_cnt;
            pb.slot_sq[o] = slot_sq;
        }
    }
}

// A packed slot block's entry: count and what is more than the common square (slot_square).
__device__ __forceinline__ void reduce_packed(const uint2 v, unsigned long long (&c)[2], unsigned long long (&more)[2]) {
    c[0] += v.x >> NARROW_SHIFT; more[0] += v.x & ((1u << NARROW_SHIFT) - 1u);
    c[1] += v.y >> NARROW_SHIFT; more[1] += v.y & ((1u << NARROW_SHIFT) - 1u);
}
__device__ __forceinline__ void reduce_wide(const ulonglong2 v, unsigned long long (&cnt)[2], unsigned long long (&t)[2]) {
    cnt[0] += v.x >> 44; t[0] += v.x & PK_MASK;
    cnt[1] += v.y >> 44; t[1] += v.y & PK_MASK;
}

// nsplit: layers whose blocks take a workgroup each.
__global__ __launch_bounds__(256) void k_reduce_parts(ProfileBuffers pb, uint32_t nsplit) {
    __shared__ unsigned long long sh_c[3][REDUCE_ENTRIES], sh_t[3][REDUCE_ENTRIES];
    constexpr uint32_t LIST = 1024;
    __shared__ uint32_t list[LIST], listed[2];
    const uint32_t lane = threadIdx.x & 63u, w = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool split = blockIdx.x < nsplit * REDUCE_BLOCKS;
    const uint32_t x = split ? blockIdx.x : blockIdx.x - nsplit * REDUCE_BLOCKS, per = split ? REDUCE_BLOCKS : REDUCE_BLOCKS / 4u;
    const ReduceLayer of = pb.reduce_layers[split ? x / per : nsplit + x / per];
    const uint32_t big = of.big, p0 = of.part0, np = of.nparts;
    // The totals over the layers that the prediction of this profile read are done with (that launch has ended), and
    // the scan that follows this one adds the new ones up: cleared here, between the two.
    if (blockIdx.x == 0u)
        for (uint32_t b = threadIdx.x; b < D1_BINS; b += 256u) pb.gprev[b] = 0ull;
    static_assert(REDUCE_ENTRIES == PART_BLOCK, "one block per block");
    unsigned long long cnt[2] = {0, 0}, t[2] = {0, 0}, zeros_sq = 0;
    if (!split) {
        const uint32_t blk = 4u * (x % per) + w, word = 1u + blk / 32u;
        const bool slot = blk >= D1_BINS / PART_BLOCK;
        // lane k has part k's head, which block it holds how
        const uint32_t* h = pb.part_head + (size_t)(p0 + min(lane, np - 1u)) * PART_HEAD;
        const bool there = h[0] != 0u && lane < np, wide = (h[word] >> (blk % 32u)) & 1u;
        const LayerState st = pb.state[big];
        const bool any = blk < (D1_BINS + st.nslots_d * D2_BINS) / PART_BLOCK;
        uint64_t wides = any ? ballot(there && wide) : 0ull, packed = any && slot ? ballot(there && !wide) : 0ull;
        if (blk == 0u) {
            if (there && wide && any) zeros_sq = pb.parts[(size_t)(p0 + lane) * PART_STRIDE + PK_ENTRIES];
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) zeros_sq += __shfl_xor(zeros_sq, d, 64);
        }
        constexpr int AT_ONCE = 8;
        while (wides) {
            ulonglong2 v[AT_ONCE];
#pragma unroll
            for (int u = 0; u < AT_ONCE; ++u) {
                v[u] = make_ulonglong2(0ull, 0ull);
                if (!wides) continue;
                v[u] = *reinterpret_cast<const ulonglong2*>(pb.parts + (size_t)(p0 + (uint32_t)__builtin_ctzll(wides)) * PART_STRIDE + blk * PART_BLOCK + 2u * lane);
                wides &= wides - 1ull;
            }
#pragma unroll
            for (int u = 0; u < AT_ONCE; ++u) reduce_wide(v[u], cnt, t);
        }
        if (packed) {
            unsigned long long c[2] = {0, 0}, more[2] = {0, 0};
            while (packed) {
                uint2 v[AT_ONCE];
#pragma unroll
                for (int u = 0; u < AT_ONCE; ++u) {
                    v[u] = make_uint2(0u, 0u);
                    if (!packed) continue;
                    v[u] = *reinterpret_cast<const uint2*>(pb.parts + (size_t)(p0 + (uint32_t)__builtin_ctzll(packed)) * PART_STRIDE + blk * PART_BLOCK + lane);
                    packed &= packed - 1ull;
                }
#pragma unroll
                for (int u = 0; u < AT_ONCE; ++u) reduce_packed(v[u], c, more);
            }
            const uint32_t bin = slot_bin_of(st, blk - D1_BINS / PART_BLOCK);
#pragma unroll
            for (uint32_t u = 0; u < 2u; ++u) {
                cnt[u] += c[u];
                t[u] += more[u] + c[u] * slot_square(bin, 2u * lane + u);
            }
        }
        reduce_store(pb, big, blk, lane, cnt, t, zeros_sq);
        return;
    }
    const uint32_t blk = x % per, word = 1u + blk / 32u;
    const uint32_t e = blk * REDUCE_ENTRIES + 2u * lane;             // and e + 1
    const bool slot = blk >= D1_BINS / PART_BLOCK;
    const LayerState st = pb.state[big];
    const uint32_t used = D1_BINS + st.nslots_d * D2_BINS;
    // which of the layer's parts hold this block, LIST of them at a time: with 64 bits an entry from the list's start,
    // packed from its end
    for (uint32_t q0 = 0; q0 < np && blk < used / PART_BLOCK; q0 += LIST) {
        __syncthreads();
        if (threadIdx.x < 2u) listed[threadIdx.x] = 0u;
        __syncthreads();
        for (uint32_t k = q0 + threadIdx.x; k < min(np, q0 + LIST); k += 256u) {
            const uint32_t* h = pb.part_head + (size_t)(p0 + k) * PART_HEAD;
            const bool there = h[0] != 0u, wide = (h[word] >> (blk % 32u)) & 1u;
            if (there && wide) list[atomicAdd(&listed[0], 1u)] = p0 + k;
            else if (there && slot) list[LIST - 1u - atomicAdd(&listed[1], 1u)] = p0 + k;
        }
        __syncthreads();
        const uint32_t n = listed[0], m = listed[1];
        // the parts four apart, four of a wave's loads at a time
        auto each = [&](uint32_t count, auto load, auto take) {
            uint32_t k = w;
            for (; k + 12 < count; k += 16) {
                const auto v0 = load(k), v1 = load(k + 4), v2 = load(k + 8), v3 = load(k + 12);
                take(v0); take(v1); take(v2); take(v3);
            }
            for (; k < count; k += 4) take(load(k));
        };
        each(n, [&](uint32_t k) { return *reinterpret_cast<const ulonglong2*>(pb.parts + (size_t)list[k] * PART_STRIDE + e); },
             [&](const ulonglong2 v) { reduce_wide(v, cnt, t); });
        if (m) {
            unsigned long long c[2] = {0, 0}, more[2] = {0, 0};
            each(m, [&](uint32_t k) { return *reinterpret_cast<const uint2*>(pb.parts + (size_t)list[LIST - 1u - k] * PART_STRIDE + blk * PART_BLOCK + lane); },
                 [&](const uint2 v) { reduce_packed(v, c, more); });
            const uint32_t bin = slot_bin_of(st, blk - D1_BINS / PART_BLOCK);
#pragma unroll
            for (uint32_t u = 0; u < 2u; ++u) {
                cnt[u] += c[u];
                t[u] += more[u] + c[u] * slot_square(bin, 2u * lane + u);
            }
        }
        if (e == 0u && w == 0u)
            for (uint32_t q = 0; q < n; ++q) zeros_sq += pb.parts[(size_t)list[q] * PART_STRIDE + PK_ENTRIES];
    }
    if (w) {
        sh_c[w - 1][2 * lane] = cnt[0]; sh_c[w - 1][2 * lane + 1] = cnt[1];
        sh_t[w - 1][2 * lane] = t[0]; sh_t[w - 1][2 * lane + 1] = t[1];
    }
    __syncthreads();
    if (w) return;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        cnt[0] += sh_c[q][2 * lane]; cnt[1] += sh_c[q][2 * lane + 1];
        t[0] += sh_t[q][2 * lane]; t[1] += sh_t[q][2 * lane + 1];
    }
    reduce_store(pb, big, blk, lane, cnt, t, zeros_sq);
}

// ---------------------------------------------------------------------------------------------
// After the pass: exact digit-1 histogram (slot bins contribute the totals of their digit-2
// bins), boundary bin per candidate, and what each boundary needs:
//   - its bin already has a slot                          -> nothing
//   - its bin is in the spilled range                     -> a slot PRE_SLOTS.. filled from the candidates
//   - it is bin 0, and that holds zeros only              -> such a slot too, filled here: the count, in digit 2 = 0
//   - neither (prediction missed), or slots run out       -> redo: exact slots, full recount
// (Four bins a thread, in whole 16-byte reads and writes.  With sixteen bins each for 256 threads, the writes to LDS, a lane's
// sixteen words apart from the next lane's, fell on four banks: 12 us on every named set, Llama's 15.5, now 8 and 11; an empty launch takes 4.5.)
constexpr uint32_t SCAN1X_THREADS = 1024;
static_assert(SCAN1X_THREADS * 4u == D1_BINS, "four bins a thread");
__global__ __launch_bounds__(SCAN1X_THREADS) void k_scan1x(ProfileBuffers pb, const uint32_t* Ktab, uint32_t J) {
    __shared__ __align__(16) uint32_t cnt[D1_BINS];
    __shared__ __align__(16) uint32_t above[D1_BINS];
    __shared__ __align__(16) double below[D1_BINS];
    __shared__ uint32_t su[16];
    __shared__ double sd[16];
    __shared__ uint32_t tbin[MAX_SLOTS];
    __shared__ __align__(16) uint8_t lut[D1_BINS];
    __shared__ uint32_t sh_redo, sh_zeros;
    __shared__ uint32_t slot_c[PRE_SLOTS];
    __shared__ unsigned long long slot_s[PRE_SLOTS];
    const uint32_t tid = threadIdx.x, big = blockIdx.x, b0 = tid * 4u;
    const uint32_t li = pb.big_layer[big];
    const LayerDesc L = pb.layers[li];
    LayerState st = pb.state[big];
    uint8_t* glut = pb.lut1 + (size_t)big * D1_BINS;
    uint8_t* glutc = pb.lutc + (size_t)big * D1_BINS;
    // this thread's four digit-1 entries and their slots: asked for now, with the slot totals below, so that the groups of
    // loads share one memory round trip instead of taking one per phase
    const uint4 craw = *reinterpret_cast<const uint4*>(pb.cnt1 + (size_t)big * D1_BINS + b0);
    const ulonglong2 s01 = *reinterpret_cast<const ulonglong2*>(pb.sq1 + (size_t)big * D1_BINS + b0);
    const ulonglong2 s23 = *reinterpret_cast<const ulonglong2*>(pb.sq1 + (size_t)big * D1_BINS + b0 + 2u);
    const uint32_t slots = *reinterpret_cast<const uint32_t*>(glut + b0);
    const uint32_t K = tid < J ? Ktab[(size_t)li * J + tid] : 0u;
    const bool spill_valid = pb.spill_over[big] == 0u;
    *reinterpret_cast<uint32_t*>(lut + b0) = slots;
    *reinterpret_cast<uint32_t*>(glutc + b0) = NO_SLOT * 0x01010101u;
    // totals of the slots the pass counted (k_reduce_parts summed them)
    static_assert(PRE_SLOTS <= SCAN1X_THREADS, "one thread per slot");
    if (tid < st.nslots_d) {
        slot_c[tid] = pb.slot_cnt[(size_t)big * SLOT_STRIDE + tid];
        slot_s[tid] = pb.slot_sq[(size_t)big * SLOT_STRIDE + tid];
    }
    if (tid == 0) sh_redo = 0u;
    __syncthreads();
    uint32_t c[4] = {craw.x, craw.y, craw.z, craw.w};
    const unsigned long long sq[4] = {s01.x, s01.y, s23.x, s23.y};
    double s[4];
    uint32_t csum = 0;
    double ssum = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t slot = slots >> (8 * k) & 0xFFu;
        unsigned long long ss = sq[k];
        if (slot != NO_SLOT) { c[k] += slot_c[slot]; ss += slot_s[slot]; }
        s[k] = sq_to_double(b0 + (uint32_t)k, ss, c[k]);
        csum += c[k];
        ssum += s[k];
    }
    if (tid == 0) sh_zeros = s[0] == 0.0 ? 1u : 0u;       // (bin 0's sum is exact: 0 only if every entry there is zero)
    // the exact histogram stays for the next profile's prediction, with its sum over the layers
    const uint4 counts = make_uint4(c[0], c[1], c[2], c[3]);
    *reinterpret_cast<uint4*>(pb.hprev + (size_t)big * D1_BINS + b0) = counts;
    *reinterpret_cast<uint4*>(cnt + b0) = counts;
    uint32_t ctot;
    const uint32_t cex = block_exclusive_scan<uint32_t>(csum, su, &ctot);
    const double sex = block_exclusive_scan<double>(ssum, sd, nullptr);
    {
        const uint32_t a0 = ctot - cex - c[0], a1 = a0 - c[1], a2 = a1 - c[2];
        *reinterpret_cast<uint4*>(above + b0) = make_uint4(a0, a1, a2, a2 - c[3]);
        const double d1 = sex + s[0], d2 = d1 + s[1];
        *reinterpret_cast<double2*>(below + b0) = make_double2(sex, d1);
        *reinterpret_cast<double2*>(below + b0 + 2u) = make_double2(d2, d2 + s[2]);
    }
    __syncthreads();
    // the sum over the layers: neighbouring lanes add to neighbouring bins (a lane adding its own bins
    // touched many cache lines per instruction, and the additions of all layers queue up on the same lines)
    for (uint32_t b = tid; b < D1_BINS; b += SCAN1X_THREADS) {
        const uint32_t cb = cnt[b];
        if (cb) atomicAdd(&pb.gprev[b], (unsigned long long)cb);
    }

    const uint32_t spill_cnt = st.spill_bin >= D1_BINS ? 0u
                             : (st.spill_bin == 0u ? ctot : above[st.spill_bin - 1u]);
    if (tid < J) {
        uint32_t bin = 0xFFFFFFFFu;
        if (K != 0u && K < L.n) {
            uint32_t lo = 0, hi = D1_BINS - 1;
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (above[mid] < K) hi = mid; else lo = mid + 1;
            }
            bin = lo;
            pb.tgt_r[(size_t)li * J + tid] = K - above[bin];
            pb.tgt_above1[(size_t)li * J + tid] = above[bin];
            pb.tgt_below[(size_t)li * J + tid] = below[bin];
            if (lut[bin] == NO_SLOT && !(spill_valid && bin >= st.spill_bin) && !(bin == 0u && sh_zeros)) atomicOr(&sh_redo, 1u);
        }
        tbin[tid] = bin;
    }
    __syncthreads();
    // Slots for the boundary bins, by the first wave: lane j holds candidate j.  Candidates ascend in
    // K, so their boundary bins never ascend and equal bins are adjacent: a run of equal bins starts
    // where the bin differs from the lane before, and its number among the runs is a prefix count.
    uint32_t bin = 0xFFFFFFFFu, pslot = NO_SLOT;
    bool valid = false, newrun = false;
    uint64_t heads_c = 0;
    if (tid < 64) {
        if (tid < J) bin = tbin[tid];
        valid = bin != 0xFFFFFFFFu;
        if (valid) pslot = lut[bin];                       // slot fixed before the pass, if any
        const uint32_t prevbin = __shfl_up(bin, 1, 64);
        newrun = valid && (tid == 0 || prevbin != bin);
        heads_c = ballot(newrun && pslot == NO_SLOT);      // runs that need a slot filled from the candidates
        if (tid == 0 && (uint32_t)__popcll(heads_c) > SLOT_STRIDE - PRE_SLOTS) sh_redo = 1u;
    }
    __syncthreads();
    const bool redo = sh_redo != 0u;
    if (redo) {
        // exact slots for every boundary bin; their digit-2 counts are recounted by a full pass
        *reinterpret_cast<uint32_t*>(glut + b0) = NO_SLOT * 0x01010101u;
        uint32_t* c2 = pb.cnt2 + (size_t)big * SLOT_STRIDE * D2_BINS;
        unsigned long long* s2 = reinterpret_cast<unsigned long long*>(pb.sq2) + (size_t)big * SLOT_STRIDE * D2_BINS;
        for (uint32_t e = tid; e < PRE_SLOTS * D2_BINS; e += SCAN1X_THREADS) { c2[e] = 0u; s2[e] = 0ull; }
        __syncthreads();
    }
    if (tid < 64) {
        const uint64_t upto = (2ull << tid) - 1ull;        // this lane and the lanes before it
        const uint64_t heads_all = ballot(newrun);
        uint32_t slot = NO_SLOT;
        if (redo) {
            if (valid) slot = (uint32_t)__popcll(heads_all & upto) - 1u;
            if (newrun) {
                glut[bin] = (uint8_t)slot;
                pb.slot_bin[(size_t)big * SLOT_STRIDE + slot] = bin;
            }
        } else if (valid) {
            if (pslot != NO_SLOT) {
                slot = pslot;
            } else {
                slot = PRE_SLOTS + (uint32_t)__popcll(heads_c & upto) - 1u;
                if (newrun) {
                    if (bin == 0u && !(spill_valid && st.spill_bin == 0u)) pb.cnt2[((size_t)big * SLOT_STRIDE + slot) * D2_BINS] = cnt[0];
                    else glutc[bin] = (uint8_t)slot;
                    pb.slot_bin[(size_t)big * SLOT_STRIDE + slot] = bin;
                }
            }
        }
        if (tid < J) pb.tgt_slot[(size_t)li * J + tid] = slot;
        if (tid == 0) {
            if (redo) atomicAdd(&pb.diag[3], 1u);
            const uint32_t nd = redo ? (uint32_t)__popcll(heads_all) : st.nslots_d;
            st.nslots_d = nd; st.nslots_t = redo ? 0u : (uint32_t)__popcll(heads_c); st.redo = redo ? 1u : 0u;
            st.spill_cnt = spill_cnt; st.spill_valid = spill_valid ? 1u : 0u;
            pb.state[big] = st;
            pb.nslots[big] = nd;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Digit-2 histograms of the slots PRE_SLOTS.. from the candidate buffer.  Four lanes per chunk: the kernel is bound
// by how many loads its waves keep in flight (eight per lane here), not by their number.
__global__ __launch_bounds__(256) void k_hist2c(ProfileBuffers pb) {
    constexpr uint32_t S = SUB_HIST;
    const SubGroup g = sub_group<S>();
    const uint32_t chunk = blockIdx.x * (256u / S) + threadIdx.x / S;
    if (chunk >= pb.nchunks_total) return;
    // what the chunk index alone addresses is fetched together; it says where the chunk's candidates are, so the
    // layer's state and the first rounds' candidates are asked for together as well
    const uint32_t big = pb.chunk_big[chunk];
    const uint32_t first = pb.chunk_first[chunk];
    const uint32_t cnt = pb.rec_cnt[chunk];
    const uint32_t start = pb.rec_start[chunk];
    materialise(big); materialise(first); materialise(cnt); materialise(start);
    if (cnt == 0u) return;
    const uint64_t base = region_start(first, big) + start;
    const LayerState st = pb.state[big];
    const uint8_t* lutc = pb.lutc + (size_t)big * D1_BINS;
    uint32_t* c2 = pb.cnt2 + (size_t)big * SLOT_STRIDE * D2_BINS;
    unsigned long long* s2 = reinterpret_cast<unsigned long long*>(pb.sq2) + (size_t)big * SLOT_STRIDE * D2_BINS;
    // Eight rounds at a time: their keys are loaded together, then their slots.  Positions past the
    // chunk's last candidate read that last candidate again (always a valid address) and are dropped.
    constexpr int AHEAD = 8;
    for (uint32_t k0 = g.sub; k0 < cnt; k0 += AHEAD * S) {
        uint32_t key[AHEAD], slot[AHEAD];
#pragma unroll
        for (int t = 0; t < AHEAD; ++t)
            key[t] = key_of(pb.tmp_x[base + min(k0 + (uint32_t)t * S, cnt - 1u)]);
        if (st.redo || st.nslots_t == 0u) return;       // (a layer without such slots: its candidates were asked for in vain)
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) slot[t] = (uint32_t)lutc[key[t] >> D1_SHIFT];
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) {
            if (slot[t] == NO_SLOT || k0 + (uint32_t)t * S >= cnt) continue;
            const uint32_t bin = key[t] >> D1_SHIFT;
            const uint32_t e = slot[t] * D2_BINS + ((key[t] >> D2_SHIFT) & (D2_BINS - 1));
            const unsigned long long s = bin ? (unsigned long long)sq_coarse(key[t]) : sq_exact(key[t]);
            atomicAdd(&c2[e], 1u);
            if (s) atomicAdd(&s2[e], s);
        }
    }
}

// The same where the slots hold many entries (the grid's smallest ratio is no small share of the layer): the additions
// queue up on the slots' few lines, so the layer that has a fair share of a workgroup's 256 chunks is counted in LDS, in
// the packed form of the streaming pass, and added to the layer's tables once; other layers' candidates go there one by
// one.  (The paper's grid, one by one and so: ResNet-18 32 and 20 us, ResNet-50 128 and 32, the GPT-2-shaped set 208 and 29,
// the Llama-shaped one 942 and 150.  Logarithmic grids from a thousandth or less: 14 to 19 and 19 to 22 us GPT-2-shaped, 17
// to 60 and 26 to 89 Llama-shaped; from more than a 512th on they need no such slots, and both kernels find nothing to do.)
constexpr uint32_t DENSE_THREADS = 1024;
constexpr uint32_t DENSE_CHUNKS = DENSE_THREADS / SUB_HIST;
constexpr uint32_t DENSE_SHARE = 64;           // chunks of one layer from which on the table in LDS pays
__global__ __launch_bounds__(DENSE_THREADS) void k_hist2c_dense(ProfileBuffers pb) {
    constexpr uint32_t S = SUB_HIST;
    __shared__ unsigned long long tab[(SLOT_STRIDE - PRE_SLOTS) * D2_BINS];     // 64 KB
    const SubGroup g = sub_group<S>();
    const uint32_t c0 = blockIdx.x * DENSE_CHUNKS, chunk = c0 + threadIdx.x / S;
    uint32_t big = 0u, first = 0u, cnt = 0u, start = 0u;
    if (chunk < pb.nchunks_total) { big = pb.chunk_big[chunk]; first = pb.chunk_first[chunk]; cnt = pb.rec_cnt[chunk]; start = pb.rec_start[chunk]; }
    materialise(big); materialise(first); materialise(cnt); materialise(start);
    // the layer of the middle chunk (any layer with more than half of the chunks is that one)
    const uint32_t c_end = min(pb.nchunks_total, c0 + DENSE_CHUNKS);
    const uint32_t main_big = pb.chunk_big[c0 + (c_end - c0) / 2u];
    const LayerState main_st = pb.state[main_big];
    const LayerDesc& ML = pb.layers[pb.big_layer[main_big]];
    const uint32_t m0 = max(c0, ML.chunk0), m1 = min(c_end, ML.chunk0 + ML.nchunks);
    const uint32_t nt = main_st.redo || m1 - m0 < DENSE_SHARE ? 0u : main_st.nslots_t;          // slots in LDS (0: none)
    for (uint32_t e = threadIdx.x; e < nt * D2_BINS; e += DENSE_THREADS) tab[e] = 0ull;
    __syncthreads();
    if (cnt != 0u) {
        const uint64_t base = region_start(first, big) + start;
        const LayerState st = pb.state[big];
        const uint8_t* lutc = pb.lutc + (size_t)big * D1_BINS;
        uint32_t* c2 = pb.cnt2 + (size_t)big * SLOT_STRIDE * D2_BINS;
        unsigned long long* s2 = reinterpret_cast<unsigned long long*>(pb.sq2) + (size_t)big * SLOT_STRIDE * D2_BINS;
        const bool in_lds = nt != 0u && big == main_big;
        constexpr int AHEAD = 8;
        for (uint32_t k0 = g.sub; k0 < cnt; k0 += AHEAD * S) {
            uint32_t key[AHEAD], slot[AHEAD];
#pragma unroll
            for (int t = 0; t < AHEAD; ++t)
                key[t] = key_of(pb.tmp_x[base + min(k0 + (uint32_t)t * S, cnt - 1u)]);
            if (st.redo || st.nslots_t == 0u) break;
#pragma unroll
            for (int t = 0; t < AHEAD; ++t) slot[t] = (uint32_t)lutc[key[t] >> D1_SHIFT];
#pragma unroll
            for (int t = 0; t < AHEAD; ++t) {
                if (slot[t] == NO_SLOT || k0 + (uint32_t)t * S >= cnt) continue;
                const uint32_t bin = key[t] >> D1_SHIFT, d2 = (key[t] >> D2_SHIFT) & (D2_BINS - 1);
                if (in_lds && bin != 0u) {
                    // (at most 256 chunks' entries: the count field holds 1023)
                    atomicAdd(&tab[(slot[t] - PRE_SLOTS) * D2_BINS + d2], PK_ONE | pk_term(key[t]));
                } else {
                    const uint32_t e = slot[t] * D2_BINS + d2;
                    const unsigned long long s = bin ? (unsigned long long)sq_coarse(key[t]) : sq_exact(key[t]);
                    atomicAdd(&c2[e], 1u);
                    if (s) atomicAdd(&s2[e], s);
                }
            }
        }
    }
    __syncthreads();
    uint32_t* c2 = pb.cnt2 + ((size_t)main_big * SLOT_STRIDE + PRE_SLOTS) * D2_BINS;
    unsigned long long* s2 = reinterpret_cast<unsigned long long*>(pb.sq2) + ((size_t)main_big * SLOT_STRIDE + PRE_SLOTS) * D2_BINS;
    for (uint32_t e = threadIdx.x; e < nt * D2_BINS; e += DENSE_THREADS) {
        const unsigned long long v = tab[e];
        if (v == 0ull) continue;
        const uint32_t n = (uint32_t)(v >> 44);
        const uint32_t bin = pb.slot_bin[(size_t)main_big * SLOT_STRIDE + PRE_SLOTS + e / D2_BINS];
        // the sums as midpoints in units of 2^16, as k_reduce_parts writes them (exponent 255: the NaN count)
        const unsigned long long s = (bin >> 4) == 255u ? (v & PK_MASK) : ((v & PK_MASK) << 8) + ((unsigned long long)n << 7);
        atomicAdd(&c2[e], n);
        if (s) atomicAdd(&s2[e], s);
    }
}

}  // namespace kimad
