// Knapsack allocation of rows that fit no LDS, in two halves (paper Appendix C; Section 3.2, Eq. optimisation).
//
// The chain of k_dp_chain_long takes a memory round trip a layer.  As in k_alloc_tree.h, the order of the sums names the same sizes
// unless two allocations lie within rounding of each other, so the layers are dealt out to two chains, both from cost 0, that run side by
// side, those that reach least first: rows are short as long as only they are in them.
//
//   k_dp_chain_long  both chains: rows 1 .. split, and rows split + 1 .. L;
//   k_dp_meet        the costs a, b of the two halves, a + b within the capacity, whose totals together are least;
//   k_dp_back        both halves back from there, side by side, every choice held against the second best.
//
// Where the second best is within rounding, anywhere, the layers are taken in their own order (k_dp_refill, k_dp_chain_long, k_dp_final,
// which otherwise leave after one load).  A size that is dearer than another of its layer and no better takes no part: the chain's
// answer is the smallest cost that attains the least total.
//
// Bound by the way of a cell from one wave to the next and by the source cells that a layer of many candidates reads.  (62 layers, 58
// thousand cells, us: one chain 135 and its way back 36; two of the layers' own order 112 and 31; two that take what reaches least first
// 86 and 24, with a meeting of 8.)
#pragma once
#include "common.h"
#include "k_alloc.h"
#include "k_alloc_chain.h"
#include "k_alloc_tree.h"

namespace kimad {

constexpr uint32_t HALVES_MAX_L = 1024, HALVES_MAX_CELLS = 131072;
constexpr uint32_t MEET_THREADS = 1024, MEET_MAX = HALVES_MAX_CELLS / MEET_THREADS;

// The halves' last rows' least values by 64 cells, and behind the first half's what the workgroups of k_dp_meet have found:
// least total, second least and where, [MEET_MAX + 1][3], and as the last the whole's with the margin.
constexpr uint32_t MEET_RESULTS = HALVES_MAX_CELLS / 64u;
static_assert(MEET_RESULTS + 3u * (MEET_MAX + 1u) <= DP_ROW_MAX, "a row of the launches by layer holds them");

__device__ __forceinline__ void f64_store_far(double* p, double v) { cell_store(p, v); }
__device__ __forceinline__ double f64_load_far(const double* p) {
    return __longlong_as_double((long long)cell_load(reinterpret_cast<const unsigned long long*>(p)));
}
// Twice what two sums of the layers' errors may differ by (k_dp_path), in every thread of a workgroup of up to sixteen waves.
__device__ __forceinline__ double rounding_margin(const double* habs, uint32_t L, double* scratch) {
    double largest = 0.0, sum = 0.0;
    for (uint32_t i = threadIdx.x; i < L; i += blockDim.x) largest += habs[i];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) largest += __shfl_xor(largest, d, 64);
    if (lane_id() == 0u) scratch[threadIdx.x >> 6] = largest;
    __syncthreads();
    for (uint32_t w = 0; w < blockDim.x / 64u; ++w) sum += scratch[w];
    __syncthreads();
    return sum < 1e300 ? sum * ((double)(L + 8u) * 0x1p-50) : DP_INF;
}
// Least value of a workgroup of sixteen waves, where it is, and the second least.
__device__ __forceinline__ Two two_of_block(const Two& mine, Two* scratch) {
    const Two t = two_wave(mine);
    if (lane_id() == 0u) scratch[threadIdx.x >> 6] = t;
    __syncthreads();
    Two all{DP_INF, DP_INF, 0u};
    if (lane_id() < blockDim.x / 64u) all = scratch[lane_id()];
    __syncthreads();
    return two_wave(all);
}

// Workgroup i: the second half's costs x = 1024 i + 0 .. 1023 at most, with the first half's a = cap - x.
__global__ __launch_bounds__(MEET_THREADS) void k_dp_meet(AllocBuffers ab, const double* __restrict__ habs, const double* __restrict__ F,
                                                          const double* __restrict__ G, const double* __restrict__ gmin, double* results) {
    constexpr uint32_t NT = MEET_THREADS, WAVES = NT / 64u;
    __shared__ double upto[NT], sg[WAVES], sl[WAVES];
    __shared__ Two s_two[WAVES];
    __shared__ uint32_t s_last;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid >> 6, cap = ab.cap, at_once = ab.flags[FLAG_AT_ONCE];
    const uint32_t x0 = blockIdx.x * NT, a_top = cap - x0;                    // (the grid ends with the capacity)
    const bool has_a = a_top + tid >= NT - 1u;
    const uint32_t a = has_a ? a_top + tid - (NT - 1u) : 0u;
    const double f = has_a ? F[a] : DP_INF, g = x0 + tid <= cap ? G[x0 + tid] : DP_INF;
    double lg = DP_INF;                                    // least of G below
    for (uint32_t w = tid; w < x0 / 64u; w += NT) lg = min_f64(lg, gmin[w]);
    if (at_once) {
        // (nothing is known of a least total, and the numbers that nobody drew are no waits given up)
        if (blockIdx.x == 0u && tid == 0u) { results[3u * MEET_MAX] = DP_INF; results[3u * MEET_MAX + 1u] = DP_INF; ab.flags[2] = 0u; }
        return;
    }
    lg = wave_min_f64(lg);
    const double in = wave_scan_min_f64(g);
    if (lane == 63u) { sg[wave] = in; sl[wave] = lg; }
    __syncthreads();
    double least = in;
    for (uint32_t w = 0; w < WAVES; ++w) {
        least = min_f64(least, sl[w]);
        if (w < wave) least = min_f64(least, sg[w]);
    }
    upto[tid] = least;
    __syncthreads();
    Two t{DP_INF, DP_INF, 0u};
    if (has_a) two_add(t, f + upto[NT - 1u - tid], a);
    t = two_of_block(t, s_two);
    if (tid == 0u) {
        f64_store_far(results + 3u * blockIdx.x, t.best);
        f64_store_far(results + 3u * blockIdx.x + 1u, t.second);
        f64_store_far(results + 3u * blockIdx.x + 2u, (double)t.at);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        s_last = atomicAdd(&ab.flags[FLAG_MET], 1u) + 1u == gridDim.x ? 1u : 0u;
    }
    __syncthreads();
    if (!s_last) return;
    t = Two{DP_INF, DP_INF, 0u};
    for (uint32_t k = tid; k < gridDim.x; k += NT) {
        const double best = f64_load_far(results + 3u * k), second = f64_load_far(results + 3u * k + 1u);
        two_add(t, best, (uint32_t)f64_load_far(results + 3u * k + 2u));
        t.second = min_f64(t.second, second);
    }
    t = two_of_block(t, s_two);
    const double margin = rounding_margin(habs, ab.L, sg);
    if (tid == 0u) {
        results[3u * MEET_MAX] = t.best;
        results[3u * MEET_MAX + 1u] = margin;
        ab.flags[FLAG_COST] = t.at;
        if (!(t.second > t.best + margin)) ab.flags[FLAG_UNSURE] = 1u;
    }
}

// The rows as k_dp_prep leaves them, for the layers in their own order.  Behind ties in a row (alloc_decided) the halves are passed over:
// k_dp_chain_long's workgroups draw no number of theirs, k_dp_meet leaves without a least total, and the rows are as k_dp_prep has left them.
// (us of all launches of the allocation, whole rows alone, behind the halves, and at once: 24 layers of 32 ratios and 4300 cells
// 56, 100, 66, 62 of 32 and 20 thousand 140, 233, 156, 161 of 5 and 58 thousand 295, 484, 326.  A word of its own for
// k_dp_chain_long to look at cost every clear allocation 1 to 13 us.)
__global__ __launch_bounds__(64) void k_dp_refill(AllocBuffers ab, double* rows, uint64_t pitch, uint32_t pad) {
    if (ab.flags[FLAG_CHAIN] == 0u) return;
    const bool as_left = ab.flags[FLAG_AT_ONCE] != 0u;
    for (uint32_t r = 1u + blockIdx.x; r <= ab.L && !as_left; r += gridDim.x)
        dp_fill_row(ab, rows, pitch, pad, r, blockIdx.y * 64u + threadIdx.x, 64u * gridDim.y);
    if (blockIdx.x == 0u && blockIdx.y == 0u && threadIdx.x == 0u) ab.flags[1] = 0u;
}

// Both halves back, a workgroup each; the one that is through last makes the outputs.  A half is walked two layers per memory round
// trip, as in k_dp_final.  `falling`: the errors (+inf: dearer than another size and no better).
constexpr uint32_t BACK_THREADS = 1024;
__global__ __launch_bounds__(BACK_THREADS) void k_dp_back(AllocBuffers ab, const double* rows, uint64_t pitch, uint32_t pad, uint32_t split,
                                                          const uint32_t* __restrict__ order, const uint32_t* __restrict__ wall, const double* __restrict__ falling,
                                                          const uint32_t* __restrict__ bad, const double* __restrict__ gmin,
                                                          const double* __restrict__ results, int32_t err_infeasible, int32_t err_nonfinite, int32_t err_internal, StepLookup sl) {
    constexpr uint32_t NT = BACK_THREADS, WAVES = NT / 64u, W_LDS = 12288;
    __shared__ uint32_t sw[W_LDS];
    __shared__ uint32_t s_cost[HALVES_MAX_L];            // the path's cost behind a row's layer
    __shared__ uint32_t s_layer[HALVES_MAX_L];
    __shared__ Two s_two[WAVES];
    __shared__ unsigned long long su64[16];
    __shared__ uint32_t s_last;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t half = blockIdx.x, i0 = half ? split : 0u, i1 = half ? ab.L : split, J = ab.J;
    const double least = results[0], margin = results[1];
    const bool there = least < DP_INF;
    // (errors so large that a half's sum may leave the doubles where the layers' own order does not: the least total says nothing)
    const bool beyond = !(margin < DP_INF);
    bool unsure = beyond;
    if (there) {
        const uint32_t n = (i1 - i0) * J;
        const bool in_lds = n <= W_LDS;
        for (uint32_t i = i0 + tid; i < i1; i += NT) s_layer[i] = order[i];
        if (in_lds)
            for (uint32_t i = i0 + wave; i < i1; i += WAVES)
                if (lane < J) sw[(i - i0) * J + lane] = wall[(size_t)order[i] * J + lane];
        uint32_t c = min(ab.flags[FLAG_COST], ab.cap);
        if (half) {
            // the second half's cost: its least total within the rest, by whole 64s and in the last of them; then within that 64
            const uint32_t rest = ab.cap - c, blocks = rest / 64u;
            const double* G = rows + (size_t)ab.L * pitch + pad;
            Two t{DP_INF, DP_INF, 0u};
            for (uint32_t b = tid; b < blocks; b += NT) two_add(t, gmin[b], b);
            const double tail = wave == WAVES - 1u && 64u * blocks + lane <= rest ? G[64u * blocks + lane] : DP_INF;
            const double tail_least = wave_min_f64(tail);
            if (wave == WAVES - 1u && lane == 0u) two_add(t, tail_least, blocks);
            t = two_of_block(t, s_two);
            if (!(t.second > t.best + margin)) unsure = true;
            const uint32_t x = 64u * t.at + lane;
            const double v = x <= rest ? G[x] : DP_INF;
            t = two_wave(Two{v, DP_INF, x});
            if (!(t.second > t.best + margin)) unsure = true;
            c = t.at;
        }
        __syncthreads();
        if (wave == 0u) {
            static_assert(KIMAD_MAX_J_CONST <= 64, "one lane per candidate");
            const uint32_t j = min(lane, J - 1u);
            auto cost = [&](uint32_t i, uint32_t k) { return in_lds ? sw[(i - i0) * J + k] : wall[(size_t)s_layer[i] * J + k]; };
            auto take = [&](uint32_t i, uint32_t k) {
                if (lane == 0u) {
                    s_cost[i] = c;
                    __hip_atomic_store(&ab.j_out[s_layer[i]], (int32_t)k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            };
            for (uint32_t i = i1; i > i0;) {
                --i;
                const uint32_t w = cost(i, j);
                const uint32_t here = ab.choice[(size_t)i * ab.stride + c];
                uint32_t before = 0u;
                if (i > i0) before = ab.choice[(size_t)(i - 1u) * ab.stride + (w <= c ? c - w : 0u)];
                const uint32_t j0 = min((uint32_t)__builtin_amdgcn_readfirstlane((int)here), J - 1u);       // (a path meets candidates only)
                take(i, j0);
                uint32_t spent = (uint32_t)__builtin_amdgcn_readlane((int)w, (int)j0);
                c = spent <= c ? c - spent : 0u;
                if (i == i0) break;
                --i;
                const uint32_t j1 = min((uint32_t)__builtin_amdgcn_readlane((int)before, (int)j0), J - 1u);
                take(i, j1);
                spent = cost(i, j1);
                c = spent <= c ? c - spent : 0u;
            }
        }
        __syncthreads();
        // what comes next at each choice
        for (uint32_t i = i0 + wave; i < i1; i += WAVES) {
            const size_t o = (size_t)s_layer[i] * J + min(lane, J - 1u);
            const uint32_t at = s_cost[i], w = lane < J ? wall[o] : 0xFFFFFFFFu;
            const double e = falling[o];
            const double val = rows[(size_t)(i + 1u) * pitch + pad + at];
            const double from = rows[(size_t)(i == i0 ? 0u : i) * pitch + pad + (w <= at ? at - w : 0u)];
            const uint64_t close = ballot(w <= at && from + e <= val + margin);
            if (close == 0ull || (close & (close - 1ull))) unsure = true;
        }
    }
    if (unsure && lane == 0u) atomicOr(&ab.flags[FLAG_UNSURE], 1u);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0u) s_last = atomicAdd(&ab.flags[FLAG_BACK], 1u) + 1u == gridDim.x ? 1u : 0u;
    __syncthreads();
    if (!s_last) return;
    unsure = __hip_atomic_load(&ab.flags[FLAG_UNSURE], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
    const int32_t j = tid < ab.L ? __hip_atomic_load(&ab.j_out[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    const bool any_bad = __syncthreads_or(tid < ab.L && bad[tid] ? 1 : 0) != 0;
    const int32_t st = any_bad ? err_nonfinite : ab.flags[2] ? err_internal : there || beyond ? 0 : err_infeasible;
    const bool chain = st == 0 && unsure;
    if (tid == 0u) {
        ab.flags[FLAG_CHAIN] = chain ? 1u : 0u;
        if (!(chain && ab.flags[FLAG_AT_ONCE])) alloc_decided(ab, chain);
        if (!chain) *ab.status = st;
    }
    if (chain) return;
    if (st != 0) {
        for (uint32_t i = tid; i < ab.L; i += NT) { ab.j_out[i] = 0; ab.K_out[i] = 0; }
        for (uint32_t i = tid; i <= ab.L; i += NT) ab.offsets_out[i] = 0;
        step_lookup(sl, NT);
        return;
    }
    static_assert(HALVES_MAX_L <= BACK_THREADS, "a thread a layer");
    const unsigned long long K = tid < ab.L ? ab.Kout[(size_t)tid * J + min((uint32_t)j, J - 1u)] : 0ull;
    unsigned long long total;
    const unsigned long long off = block_exclusive_scan<unsigned long long>(K, su64, &total);
    if (tid < ab.L) { ab.j_out[tid] = j; ab.K_out[tid] = K; ab.offsets_out[tid] = off; }     // (j stored again: the look-up reads it through the caches)
    if (tid == 0u) ab.offsets_out[ab.L] = total;
    step_lookup(sl, NT);
}

}  // namespace kimad
