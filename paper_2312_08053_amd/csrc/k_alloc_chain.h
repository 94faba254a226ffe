// The allocation's recurrence by workgroups that run side by side, each with its own cost cells (paper Appendix C).
//
// A layer's row needs nothing but the cells at or below its own of the row before.  So workgroup b keeps cells
// [b W, (b + 1) W) through all the layers: the first one depends on nobody and runs ahead, the others follow at a
// distance, and a layer is no longer a sweep of one compute unit over the whole row, nor a launch.
//
// A row's cells travel through memory and stand for themselves: k_dp_prep fills the rows with ROW_EMPTY, a bit pattern
// that no total has (a total is a number or +inf: a minimum taken from +inf on is never a NaN), a workgroup stores each
// cell once with a device-scope store, and a reader that finds ROW_EMPTY asks again.  There is no flag, and no order
// between two stores matters.
//
// (One workgroup sweeping whole rows, bound by one compute unit's LDS, and a launch per layer where a row fits no LDS took,
// against these: 148 layers of 999 cells 125 and 61 us, 161 layers of 996 cells 117 and 62; 62 layers with the exact cost
// axis, 12 thousand cells 249 and 72, 58 thousand 395 and 149, 130 thousand with 64 candidates 702 and 374, 480 thousand 892
// and 743.)
//
// Progress.  A workgroup takes its number b from a counter when it starts, so all lower numbers belong to workgroups
// that are already running, and it waits for lower numbers only: the lowest unfinished one never waits for long,
// however few of the others fit on the chip.  A wait is given up after CHAIN_POLLS reads (seconds), which the walk
// back reports as an internal error.  A wave that has given up waits no more, in this row or a later one, and the loaders of
// k_dp_chain look every CHAIN_LOOK reads whether one has: the launch ends after a few such waits, however many layers are
// left.  A number beyond the grid, as calls that share one set of tables and overlap hand out, owns no cells: its workgroup
// leaves, and the call reports an internal error too.  (The workgroups that look after a piece of the layers have the highest
// numbers and wait for the ones that keep cells; nobody waits for them.)
#pragma once
#include "common.h"
#include "k_alloc.h"

namespace kimad {

constexpr uint32_t CHAIN_POLLS = 1u << 22, CHAIN_LOOK = 1u << 12;

__device__ __forceinline__ unsigned long long cell_load(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void cell_store(double* p, double v) {
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool cell_empty(unsigned long long v) { return (uint32_t)(v >> 32) == 0xFFFFFFFFu; }

// Whether a wait of `polls` reads goes on (the same in all lanes).
__device__ __forceinline__ bool wait_on(const AllocBuffers& ab, uint32_t polls) {
    if (polls > ab.polls) {
        if (lane_id() == 0) atomicAdd(&ab.flags[2], 1u);
        return false;
    }
    return __builtin_amdgcn_readfirstlane(__hip_atomic_load(&ab.flags[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0u;
}

// Least value over the four 16-lane rows of a wave, in every row (min is exact: the order does not matter).
__device__ __forceinline__ double min_over_rows(double v) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    {
        const uint32_t lo = (uint32_t)__double2loint(v), hi = (uint32_t)__double2hiint(v);
        const u32x2 a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false), b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        v = min_f64(__hiloint2double((int)b.x, (int)a.x), __hiloint2double((int)b.y, (int)a.y));
    }
    const uint32_t lo = (uint32_t)__double2loint(v), hi = (uint32_t)__double2hiint(v);
    const u32x2 a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false), b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return min_f64(__hiloint2double((int)b.x, (int)a.x), __hiloint2double((int)b.y, (int)a.y));
}

// The value of another lane inside groups of 2, 4, 8 or 16 neighbouring lanes, through DPP moves (a shuffle goes
// through the LDS crossbar: a dependent round trip per step).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
// Least value of a wave, in every lane.
__device__ __forceinline__ double wave_min_f64(double v) {
    v = min_f64(v, dpp_f64<0xB1>(v));                      // quad_perm [1,0,3,2]
    v = min_f64(v, dpp_f64<0x4E>(v));                      // quad_perm [2,3,0,1]
    v = min_f64(v, dpp_f64<0x141>(v));                     // row_half_mirror
    v = min_f64(v, dpp_f64<0x140>(v));                     // row_mirror
    return min_over_rows(v);
}

// ---- rows that fit LDS -------------------------------------------------------------------------
// A compute wave looks after sixteen cells, the same ones in each of its four 16-lane rows; lane 16 r + k holds list record
// 4 k + r and hands it to its row by DPP, so the four rows share a layer's records and a minimum over the rows closes
// the layer.  The workgroup's previous row is in LDS up to its own last cell: its own cells from its compute waves, the lower
// ones from memory, brought by other waves: CHAIN_LOADERS groups of them take the rows in turn, each asking for its next row
// when it has put down one, so that a row is asked for CHAIN_LOADERS layers before it is needed, and a wave that waits
// for memory waits for its own row only; one more wave brings the layers' records.  One barrier a layer.
// Bound by the chain barrier, LDS read, four fp64 additions, minimum over the rows, LDS write: 0.22 us a layer in the first
// workgroup, and 1 to 2 us that each workgroup starts behind the one below it.  (The compute waves wait for no memory at
// all: with the records asked for by them, and the cells' stores in the same queue, a layer took 0.4 us.  148 layers of
// 999 cells: one loader wave a group 71 us, two 61, four 62; four groups of one wave 91.
// Few layers want few workgroups, each of which starts behind the one below, many a short layer: all launches of the
// allocation with rows of 1001 cells, 64 ratios and four or eight waves, 20 layers 32.9 and 30.7 us, 60 55.9 and 52.3, 128 78.6 and 76.5,
// 161 89.8 and 88.5, 218 107.9 and 108.9, 300 134.7 and 138.5, 500 198 and 210, 1000 357 and 386; with 16 ratios 60 47.8 and
// 44.0, 148 73.6 and 72.1, 300 118 and 122.  With 2001 cells the two are the same (60 layers 86.1 and 86.0, 148 169.8 and 169.7, 300 214.7
// and 213.4).  Rows beyond 2048 cells take four, whose loaders leave no room for eight: 60 layers of 4097 cells 126 and, with three
// waves a loader group, 192, 148 layers 244 and 396.)
constexpr uint32_t CHAIN_NARROW_L = 192;        // layers beyond which four waves look after rows of up to 1024 cells
constexpr uint32_t CHAIN_LOADERS = 2;
constexpr uint32_t CHAIN_RECS = 4;              // layers whose records are in LDS, and under way from memory
static_assert(CHAIN_RECS % 2 == 0, "the rows change places every layer");

// Minimum over the records of the lane's row, of which there are at most 4 B.  All cells are asked for before the first is
// used.  (`then`: what is asked for behind them.)
template <int K4, int B>
__device__ __forceinline__ void chain_ask(uint32_t neg_cost, uint32_t prev, double (&t)[B][4]) {
    uint32_t q[4];
    row_addr_sub4<4 * K4>(prev, neg_cost, q);
#pragma unroll
    for (int u = 0; u < 4; ++u) t[K4][u] = *(lds_cdouble_ptr)(uintptr_t)q[u];
}
template <int B, typename F>
__device__ __forceinline__ double chain_records(uint32_t neg_cost, double err, double one, uint32_t prev, F then) {
    double t[B][4], m[B];
    chain_ask<0>(neg_cost, prev, t);
    if constexpr (B > 1) chain_ask<1>(neg_cost, prev, t);
    if constexpr (B > 2) chain_ask<2>(neg_cost, prev, t);
    if constexpr (B > 3) chain_ask<3>(neg_cost, prev, t);
    then();
    acc_rec_error4<0>(t[0], err, one);
    if constexpr (B > 1) acc_rec_error4<4>(t[1], err, one);
    if constexpr (B > 2) acc_rec_error4<8>(t[2], err, one);
    if constexpr (B > 3) acc_rec_error4<12>(t[3], err, one);
#pragma unroll
    for (int k = 0; k < B; ++k) m[k] = min_f64(min_f64(t[k][0], t[k][1]), min_f64(t[k][2], t[k][3]));
    double best = m[0];
    if constexpr (B > 1) best = min_f64(best, m[1]);
    if constexpr (B > 2) best = min_f64(best, m[2]);
    if constexpr (B > 3) best = min_f64(best, m[3]);
    return min_f64(best, DP_INF);                 // (never a NaN: a cell holds a number or ROW_EMPTY)
}

// The layers, for one compute wave.  CELLS: cells of the workgroup, and of +inf before cost 0 of its rows.
template <uint32_t CELLS>
__device__ __forceinline__ void chain_compute(uint32_t layers, double* rows_g, uint32_t rstride, uint32_t c0, uint32_t wave, double* row_a,
                                              double* row_b, const uint4 (*recs)[64]) {
    const uint32_t lane = lane_id(), c = c0 + wave * 16u + (lane & 15u);
    double one = 1.0;
    asm volatile("" : "+v"(one));          // keep 1.0 in a vector register pair
    double* out = rows_g + rstride + c;
    uint4 R = recs[0][lane];
    for (uint32_t i0 = 0; i0 < layers; i0 += CHAIN_RECS) {
#pragma unroll
        for (uint32_t u = 0; u < CHAIN_RECS; ++u) {
            if (i0 + u >= layers) break;
            const uint32_t at = lds_addr(((u & 1u) ? row_b : row_a) + CELLS + c);
            const uint32_t neg = R.z, n = (uint32_t)__builtin_amdgcn_readfirstlane(R.w);
            const double err = rec_err(R);
            auto next = [&]() { R = recs[(u + 1u) % CHAIN_RECS][lane]; };
            double best;
            if (n <= 16u) best = chain_records<1>(neg, err, one, at, next);
            else if (n <= 32u) best = chain_records<2>(neg, err, one, at, next);
            else if (n <= 48u) best = chain_records<3>(neg, err, one, at, next);
            else best = chain_records<4>(neg, err, one, at, next);
            best = min_over_rows(best);
            if (lane < 16u) {
                ((u & 1u) ? row_a : row_b)[CELLS + c] = best;
                cell_store(out, best);
            }
            out += rstride;
            lds_barrier();
        }
    }
}

// The records that any cell of this workgroup can afford (the first ones: costs ascend, an unused record costs 0xFFFFFFFF),
// for one wave: layer i + 2 is put down in layer i, for the compute waves to read in layer i + 1.
struct ChainRecords {
    const AllocBuffers& ab;
    const DpLists& dl;
    uint32_t c_hi;
    uint4 (*recs)[64];
    uint32_t rw[CHAIN_RECS];
    double re[CHAIN_RECS];

    __device__ __forceinline__ void ask(uint32_t i, uint32_t& w, double& e) {
        const uint32_t rec = (lane_id() & 15u) * 4u + (lane_id() >> 4);
        const size_t o = (size_t)min(i, ab.L - 1u) * ab.J + min(rec, ab.J - 1u);
        w = rec < ab.J ? dl.w[o] : 0xFFFFFFFFu;
        e = dl.e[2 * o];
    }
    __device__ __forceinline__ void put(uint32_t slot, uint32_t w, double e) {
        const bool can = w <= c_hi;
        const uint32_t n = (uint32_t)__popcll(ballot(can));
        const double x = can ? e : DP_INF;
        recs[slot][lane_id()] = make_uint4((uint32_t)__double2loint(x), (uint32_t)__double2hiint(x), can ? 0u - 8u * w : 0u, n);
    }
    __device__ __forceinline__ void start() {
#pragma unroll
        for (uint32_t a = 0; a < CHAIN_RECS; ++a) ask(a, rw[a], re[a]);
        put(0u, rw[0], re[0]);
        put(1u, rw[1], re[1]);
#pragma unroll
        for (uint32_t a = 0; a < 2u; ++a) ask(CHAIN_RECS + a, rw[a], re[a]);
    }
    __device__ __forceinline__ void run() {
        for (uint32_t i0 = 0; i0 < ab.L; i0 += CHAIN_RECS) {
#pragma unroll
            for (uint32_t u = 0; u < CHAIN_RECS; ++u) {
                if (i0 + u >= ab.L) break;
                constexpr uint32_t A = CHAIN_RECS;
                put((u + 2u) % A, rw[(u + 2u) % A], re[(u + 2u) % A]);
                ask(i0 + u + 2u + A, rw[(u + 2u) % A], re[(u + 2u) % A]);
                lds_barrier();
            }
        }
    }
};

// The lower cells of rows g + 1, g + 1 + CHAIN_LOADERS, ..., for one wave of a loader group: cells first, first + 64 GW, ...
template <int M, uint32_t GW, uint32_t CELLS>
__device__ __forceinline__ void chain_load(const AllocBuffers& ab, const double* rows_g, uint32_t rstride, uint32_t c0, uint32_t g,
                                           uint32_t first, double* row_a, double* row_b) {
    constexpr uint32_t N = CHAIN_LOADERS;
    unsigned long long v[M];
    // (a row beyond the last: the last one again, not used)
    auto ask = [&](uint32_t r) {
        const unsigned long long* row = reinterpret_cast<const unsigned long long*>(rows_g + (size_t)min(r, ab.L) * rstride);
#pragma unroll
        for (int m = 0; m < M; ++m) v[m] = cell_load(row + min(first + (uint32_t)m * 64u * GW, c0 - 1u));
    };
    auto any_empty = [&]() {
        uint32_t top = 0u;                            // (an empty cell has the greatest high word)
#pragma unroll
        for (int m = 0; m < M; ++m) top = max(top, (uint32_t)(v[m] >> 32));
        return ballot(top == 0xFFFFFFFFu) != 0ull;
    };
    ask(g + 1u);
    uint32_t limit = min(ab.polls, CHAIN_LOOK);       // reads of a wait before the next look; 0: given up
    uint32_t i = 0;                                   // layers whose barrier is behind us
    for (; i < min(g, ab.L); ++i) lds_barrier();
    static_assert(N % 2 == 0, "a group's rows all go to the same half of LDS");
    double* dst = ((g & 1u) ? row_a : row_b) + CELLS;
    while (i < ab.L) {
        uint32_t polls = 0;
        while (any_empty()) {
            if (__builtin_expect(++polls > limit, 0)) {
                if (limit == 0u || !wait_on(ab, polls)) {
                    limit = 0u;
                    break;
                }
                limit = polls + CHAIN_LOOK;
            }
            asm volatile("" ::: "memory");
            ask(i + 1u);
        }
#pragma unroll
        for (int m = 0; m < M; ++m) dst[min(first + (uint32_t)m * 64u * GW, c0 - 1u)] = __longlong_as_double((long long)v[m]);
        ask(i + 1u + N);
        for (uint32_t k = 0; k < N && i < ab.L; ++k, ++i) lds_barrier();
    }
}

// ---- which candidate won, and where it came from ------------------------------------------------
// While the chain goes on, further workgroups of its launch follow the rows as they come, a piece of the layers each, in
// which every cell finds its winning candidate (in list order with a strict "<", then the lowest member of the winner's run
// whose rounded total is the same) and is then followed down to the piece's first row.  What is left for k_dp_walk is one
// step a piece, not one a layer, and when the chain ends the rows of all but the last pieces have been dealt with.
// Bound by the vector instructions per cell and candidate: a layer takes a workgroup several times as long as the chain.
// What the last ones take is added to the chain's time, so the last layers are pieces of their own (Pieces, k_alloc.h), and
// have a workgroup for every BLOCK_CELLS of their cells.  (us, with a launch of one workgroup per layer and 256 cells after the
// chain and a walk of one step a layer, and now.  148 layers of 999 cells: chain 59, choice 8, walk 18; chain 64, walk 10.  62
// layers with up to 50 candidates: 31, 10 and 12; 38 and 9.  All launches of the allocation, 64 ratios: 20 layers 36 and 31, 500
// 230 and 197, 1000 421 and 357; 148 layers of 4097 cells 260 and 245.)
// (Blocks of 128, 256 and 512 cells, us: all launches of the allocation, 20 layers 30.3, 30.5, 31.0, 148 84.2, 84.0, 84.0; the chain in
// the steps of ResNet-18 with 50 ratios 40.8, 41.5, 41.7, of the GPT-2-shaped set 65.4, 65.5, 65.9; that set's round with the allocation
// beside it, whose kernels go without the compute units that wait here, 415, 404, 400.)
constexpr uint32_t BLOCK_CELLS = 256;

struct PieceList {
    double e_before[KIMAD_MAX_J_CONST];
    uint32_t w[KIMAD_MAX_J_CONST], jj[KIMAD_MAX_J_CONST];
};

// Cells [lo, hi] of layers [first, first + m) for one workgroup of NT threads (m > 1: all cells).  rows: two rows in LDS, `pitch`
// cells apart, a cell before each.
template <uint32_t MAXC, uint32_t NT>
__device__ __forceinline__ void chain_choose(const AllocBuffers& ab, const DpLists& dl, const double* rows_g, uint32_t rstride, uint32_t first,
                                             uint32_t m, uint32_t piece, uint32_t lo, uint32_t hi, double* rows, uint32_t pitch, PieceList* lists,
                                             uint16_t (*src)[MAXC], uint8_t (*win)[MAXC]) {
    constexpr uint32_t CPT = (MAXC + NT - 1u) / NT, U = CPT <= 2u ? 8u : CPT <= 3u ? 4u : 2u;     // candidates whose cells are asked for together (four of five cells spill)
    const uint32_t tid = threadIdx.x, lane = lane_id();
    const uint32_t mine = lo + (uint32_t)__builtin_amdgcn_readfirstlane(tid & ~63u);   // the wave's first cell: none beyond hi
    unsigned long long v[CPT];
    auto ask = [&](uint32_t i) {
        const unsigned long long* row = reinterpret_cast<const unsigned long long*>(rows_g + (size_t)i * rstride);
#pragma unroll
        for (uint32_t q = 0; q < CPT; ++q) v[q] = cell_load(row + min(tid + q * NT, hi));
    };
    auto any_empty = [&]() {
        uint32_t top = 0u;
#pragma unroll
        for (uint32_t q = 0; q < CPT; ++q) top = max(top, (uint32_t)(v[q] >> 32));
        return ballot(top == 0xFFFFFFFFu) != 0ull;
    };
    uint32_t limit = min(ab.polls, CHAIN_LOOK);       // as in chain_load; but a wait given up is counted if it is the first one
    uint32_t polls = 0;
    auto go_on = [&]() {
        if (__builtin_expect(++polls > limit, 0)) {
            if (limit && polls > ab.polls && lane == 0) atomicCAS(&ab.flags[2], 0u, 1u);
            if (limit == 0u || polls > ab.polls ||
                __builtin_amdgcn_readfirstlane(__hip_atomic_load(&ab.flags[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0u) {
                limit = 0u;
                return false;
            }
            limit = min(ab.polls, polls + CHAIN_LOOK);
        }
        return true;
    };
    // one wave waits for the first row's last cell, with pauses: a piece may have to wait for most of the chain
    if (tid < 64u) {
        const unsigned long long* cell = reinterpret_cast<const unsigned long long*>(rows_g + (size_t)first * rstride) + hi;
        while (cell_empty(cell_load(cell)) && go_on()) __builtin_amdgcn_s_sleep(8);
    }
    __syncthreads();
    ask(first);
    for (uint32_t s = 0; s < m; ++s) {
        const uint32_t i = first + s;
        PieceList& list = lists[s & 1u];
        double* prev = rows + (s & 1u) * pitch + 1u;
        const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane(dl.n[i]);
        // lane k of every wave holds list record k (one that is not there costs more than any cell can pay)
        const size_t o = (size_t)i * ab.J + min(lane, ab.J - 1u);
        const uint32_t my_w = dl.w[o];
        const int my_w8 = lane < n ? (int)(8u * my_w) : 0x3FFFFFFF;
        const double my_e = lane < n ? dl.e[2 * o] : DP_INF;
        if (tid < n) {
            list.w[tid] = my_w; list.jj[tid] = dl.jj[o];
            list.e_before[tid] = dl.e[2 * o + 1];
        }
        polls = 0;
        while (any_empty() && go_on()) {
            asm volatile("" ::: "memory");
            ask(i);
        }
#pragma unroll
        for (uint32_t q = 0; q < CPT; ++q)
            if (tid + q * NT < MAXC) prev[tid + q * NT] = __longlong_as_double((long long)v[q]);
        if (tid == 0) prev[-1] = DP_INF;
        if (s + 1u < m) ask(i + 1u);
        lds_barrier();
        const int before = (int)lds_addr(prev) - 8;      // the cell of +inf, for what a cell cannot afford
        // NQ cells a thread, NT apart
        auto choose = [&](auto nq) {
            constexpr uint32_t NQ = decltype(nq)::value;
            double best[NQ];
            uint32_t bk[NQ];
            int at[NQ];
#pragma unroll
            for (uint32_t q = 0; q < NQ; ++q) { best[q] = DP_INF; bk[q] = 0xFFu; at[q] = before + 8 + 8 * (int)min(lo + tid + q * NT, hi); }
            for (uint32_t k0 = 0; k0 < n; k0 += U) {
                double t[U][NQ];
#pragma unroll
                for (uint32_t u = 0; u < U; ++u) {
                    const int w8 = __builtin_amdgcn_readlane(my_w8, (int)(k0 + u));
#pragma unroll
                    for (uint32_t q = 0; q < NQ; ++q) t[u][q] = *(lds_cdouble_ptr)(uintptr_t)(uint32_t)max(at[q] - w8, before);
                }
#pragma unroll
                for (uint32_t u = 0; u < U; ++u) {
                    const double e = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(my_e), (int)(k0 + u)),
                                                      __builtin_amdgcn_readlane(__double2loint(my_e), (int)(k0 + u)));
#pragma unroll
                    for (uint32_t q = 0; q < NQ; ++q) {
                        const double x = t[u][q] + e;
                        bk[q] = x < best[q] ? k0 + u : bk[q];
                        best[q] = min_f64(x, best[q]);
                    }
                }
            }
#pragma unroll
            for (uint32_t q = 0; q < NQ; ++q) {
                const uint32_t c = lo + tid + q * NT;
                if (c > hi) continue;
                uint32_t bj = 0xFFu, from = 0xFFFFu;
                if (bk[q] != 0xFFu) {
                    // Only the winner's run matters: if the member before its last one rounds to the same total
                    // (never for a single: that error is NaN), the lowest such member wins.
                    const uint32_t jj = list.jj[bk[q]];
                    bj = jj >> 8;
                    from = c - list.w[bk[q]];
                    const double p = prev[from];
                    if (p + list.e_before[bk[q]] == best[q]) {
                        const uint32_t jlo = jj & 0xFFu;
                        uint32_t j = bj - 1u;
                        while (j > jlo && p + ab.E[(size_t)i * ab.J + j - 1] == best[q]) --j;
                        bj = j;
                    }
                }
                win[s][c] = (uint8_t)bj;
                src[s][c] = (uint16_t)from;
            }
        };
        if (mine + NT <= hi) choose(std::integral_constant<uint32_t, CPT>{});
        else if (mine <= hi) choose(std::integral_constant<uint32_t, 1u>{});
    }
    __syncthreads();
    for (uint32_t c = lo + tid; c <= hi; c += NT) {
        uint32_t at = c;
        uint8_t* to = ab.choice + (size_t)first * ab.stride + (size_t)c * m;
        for (uint32_t s = m; s-- > 0u;) {
            to[s] = win[s][at];
            at = min((uint32_t)src[s][at], ab.cap);            // (a feasible path never meets the 0xFFFF of an empty cell)
        }
        ab.cprev[(size_t)piece * ab.stride + c] = (uint16_t)at;
    }
}

// W: compute waves, GW: waves of a loader group, MAXC: cells of the longest row.  The first `keepers` numbers keep cells, the
// others look after a piece each.
constexpr uint32_t chain_threads(uint32_t w, uint32_t gw) { return 64u * (w + 1u + CHAIN_LOADERS * gw); }
template <uint32_t MAXC, uint32_t W, uint32_t GW>
__global__ __launch_bounds__(chain_threads(W, GW)) void k_dp_chain(AllocBuffers ab, DpLists dl, double* __restrict__ rows_g, uint32_t rstride,
                                                                   uint32_t keepers, const uint32_t* __restrict__ gate) {
    if (gate && *gate == 0u) return;               // (decided: k_dp_path)
    constexpr uint32_t NT = chain_threads(W, GW), CELLS = 16u * W;
    static_assert(MAXC % CELLS == 0, "whole workgroups");
    __shared__ double rows[2][CELLS + MAXC];       // CELLS cells of +inf before cost 0: a record costs at most c_hi here
    __shared__ uint4 recs[CHAIN_RECS][64];
    __shared__ PieceList lists[2];
    __shared__ uint16_t src[Pieces::MOST][MAXC];
    __shared__ uint8_t win[Pieces::MOST][MAXC];
    __shared__ uint32_t sh_b;
    const uint32_t tid = threadIdx.x;
    if (tid == 0) sh_b = atomicAdd(&ab.flags[1], 1u);
    __syncthreads();
    const uint32_t number = (uint32_t)__builtin_amdgcn_readfirstlane(sh_b);
    if (number >= gridDim.x) {
        if (tid == 0) atomicAdd(&ab.flags[2], 1u);
        return;
    }
    if (number >= keepers) {
        const Pieces pieces(ab.L);
        const uint32_t blocks = ab.cap / BLOCK_CELLS + 1u, x = number - keepers;
        const uint32_t p = x < pieces.fours ? x : pieces.fours + (x - pieces.fours) / blocks, first = pieces.first(p);
        const uint32_t lo = x < pieces.fours ? 0u : (x - pieces.fours) % blocks * BLOCK_CELLS;
        chain_choose<MAXC, NT>(ab, dl, rows_g, rstride, first, pieces.first(p + 1u) - first, p, lo,
                               x < pieces.fours ? ab.cap : min(lo + BLOCK_CELLS - 1u, ab.cap), rows[0], CELLS + MAXC, lists, src, win);
        return;
    }
    const uint32_t c0 = number * CELLS;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    for (uint32_t x = tid; x < 2u * CELLS + c0; x += NT) {
        rows[0][x] = x == CELLS ? 0.0 : DP_INF;
        rows[1][x] = DP_INF;
    }
    if (wave == W) {
        ChainRecords cr{ab, dl, c0 + CELLS - 1u, recs};
        cr.start();
        __syncthreads();
        cr.run();
        return;
    }
    __syncthreads();
    if (wave < W) {
        chain_compute<CELLS>(ab.L, rows_g, rstride, c0, wave, rows[0], rows[1], recs);
        return;
    }
    const uint32_t load = wave - W - 1u, g = load / GW, first = load % GW * 64u + lane_id();
    const uint32_t m = (c0 + 64u * GW - 1u) / (64u * GW);
    constexpr uint32_t MOST = (MAXC + 64u * GW - 1u) / (64u * GW);
    if (m == 0u) {
        for (uint32_t i = 0; i < ab.L; ++i) lds_barrier();
    } else if (m <= 4u) {
        chain_load<4, GW, CELLS>(ab, rows_g, rstride, c0, g, first, rows[0], rows[1]);
    } else if (MOST <= 8u || m <= 8u) {
        chain_load<8, GW, CELLS>(ab, rows_g, rstride, c0, g, first, rows[0], rows[1]);
    } else {
        chain_load<(int)(MOST > 8u ? MOST : 8u), GW, CELLS>(ab, rows_g, rstride, c0, g, first, rows[0], rows[1]);
    }
}

// ---- rows too long for LDS ----------------------------------------------------------------------
// Every wave is on its own with 64 cells, one a lane, and reads every source cell from memory, all of a layer's together.
// CHAIN_PAD cells of +inf stand before cost 0.  SETS: sixteens of candidates; lane 16 r + k holds candidates k, k + 16, ... and
// hands them to its row by DPP.  The total is stored as soon as it is known; which candidate it came from (the first one in
// order that attains it) is looked for while the store is under way.  Bound by the way of a cell from one wave to the next
// (store, poll, load: about 1 us) and, on long rows, by the source cells read (58 thousand cells, 32 candidates: 15 MB a
// layer, 2.3 us).  With more than sixteen candidates the cheapest four's cells are waited for before all are asked for
// through the caches (149 against 160 us with device-scope loads for all; with sixteen or fewer the wait costs more than it
// saves, 83 against 72).  Sixteen cells a wave, the candidates shared by its four rows, read twice the lines: 190.
// Two waves a workgroup, whose source cells lie close together, share what its compute unit's cache holds, and are half as many workgroups
// to start one behind the other; but they share its paths, so that a layer takes longer, the more the more candidates it has: worth it
// where the row is long for the layers, on any row from 90112 cells on, and for halves.  (us of all launches of the allocation, workgroups of one
// wave and of two, layers of 16 candidates: 2 layers 8 thousand cells 19 and 18, 58 thousand 36 and 31; 6 layers 8 thousand 24 and 24, 10.5
// 25 and 25, 13.5 26 and 25, 58 45 and 40; 20 layers 13.5 44 and 46, 17 47 and 47, 22 51 and 51, 58 76 and 73; 62 layers 13.5
// 99 and 107, 28 120 and 118, 58 146 and 151, 95 182 and 180.  Of 64: 2 layers 8 thousand cells 22 and 22, 13.5 23 and 23; 8 layers 13.5 38 and 40, 17
// 40 and 41, 22 43 and 42, 58 64 and 60; 15 layers 22 64 and 64, 46 81 and 86, 74 105 and 102; 161 layers 4300 cells 385 and 448, 58 thousand
// 608 and 615, 74 678 and 719, 95 747 and 736, 120 994 and 882.  By halves 62 layers of 32 and 4300 cells 85 and 90, 13 thousand 96 and 93, 58 125
// and 122, 131 177 and 168; 161 of 64 236 and 247, 259 and 260, 326 and 354, 432 and 461; 30 of 5 and 58 thousand 76 and 67.)
constexpr uint32_t CHAIN_PAD = 64;
constexpr uint32_t CHAIN_LONG_WAVES = 2;             // of a workgroup, at most
inline uint32_t chain_long_waves(uint64_t L, uint64_t J, uint64_t cells) {
    const bool short_lists = J <= 16;
    return cells >= 90112u || (L <= (short_lists ? 30u : 15u) && cells >= 8192u + (short_lists ? 512u : 1024u) * L) ? CHAIN_LONG_WAVES : 1u;
}

// Two halves of the layers side by side (k_alloc_halves.h), each from cost 0, every range of cells by two workgroups of neighbouring
// numbers; or, where order is null, all layers one after another, if `gate` (optional) says so.
struct ChainHalves {
    const uint32_t* order;             // [L] the layers, the first half's and then the second's
    const double* falling;             // [L][J] their errors
    double* least[2];                  // [cells / 64] least values of the halves' last rows
    uint32_t split;                    // layers of the first half
    const uint32_t* gate;
};

// PAIR: two waves a workgroup, which may be in halves.  (What only halves need costs workgroups of one wave up to a tenth: 161 layers of 32
// candidates and 9 thousand cells 296 -> 326 us.  Two waves are the faster for it, and for `order` looked at as the kernel runs: 8 layers
// of 131 thousand cells and 64 candidates take 92 us and 95 without, halves of 161 layers and 58 thousand cells 354 and 361.)
template <int SETS, bool PAIR>
__global__ __launch_bounds__(PAIR ? 64u * CHAIN_LONG_WAVES : 64u) void k_dp_chain_long(AllocBuffers ab, const uint32_t* __restrict__ wall, double* rows, uint64_t pitch,
                                                                 ChainHalves ch) {
    const uint32_t lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (ch.gate && *ch.gate == 0u) return;
    __shared__ uint32_t sh_number;
    if (threadIdx.x == 0u) sh_number = atomicAdd(&ab.flags[1], 1u);
    __syncthreads();
    const uint32_t number = (uint32_t)__builtin_amdgcn_readfirstlane(sh_number);
    if (number >= gridDim.x) {
        if (threadIdx.x == 0u) atomicAdd(&ab.flags[2], 1u);
        return;
    }
    const bool halves = PAIR && ch.order != nullptr;
    const uint32_t half = halves ? number & 1u : 0u;
    const uint32_t c0 = (halves ? number >> 1 : number) * blockDim.x + 64u * wave, c = c0 + lane, c_hi = c0 + 63u;
    if (c0 > ab.cap) return;
    uint32_t i0 = half ? ch.split : 0u;
    const uint32_t first = i0, i1 = halves && !half ? ch.split : ab.L;
    const double* __restrict__ E = halves ? ch.falling : ab.E;
    auto layer = [&](uint32_t i) { return halves ? ch.order[min(i, ab.L - 1u)] : min(i, ab.L - 1u); };
    double one = 1.0;
    asm volatile("" : "+v"(one));
    bool gave_up = false;
    if (halves) {
        // rows that do not reach these cells yet
        uint32_t reach = 0u, skip = 0u;
        for (uint32_t p = first; p < i1; p += 64u) {
            const uint32_t i = p + lane, w = i < i1 ? min(wall[(size_t)layer(i) * ab.J + ab.J - 1u], ab.cap + 1u) : 0u;
            const uint32_t upto = reach + wave_scan_add_u32(w);
            skip += (uint32_t)__popcll(ballot(i < i1 && upto < c0));
            reach = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
        }
        for (; skip; --skip, ++i0) {
            cell_store(rows + (size_t)(i0 + 1u) * pitch + CHAIN_PAD + c, DP_INF);
            ab.choice[(size_t)i0 * ab.stride + c] = 0xFFu;
        }
    }
    uint32_t w_next[SETS];
    double e_next[SETS];
    auto ask_records = [&](uint32_t i) {
        const size_t o0 = (size_t)layer(i) * ab.J;
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            const uint32_t k = 16u * (uint32_t)s + (lane & 15u);
            const size_t o = o0 + min(k, ab.J - 1u);
            w_next[s] = k < ab.J ? wall[o] : 0xFFFFFFFFu;
            e_next[s] = E[o];
        }
    };
    ask_records(i0);
    double last = DP_INF;
    for (uint32_t i = i0; i < i1; ++i) {
        // a candidate that no cell here can afford reads the cells before cost 0
        uint32_t n = 0, neg[SETS];
        double err[SETS];
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            const bool can = w_next[s] <= c_hi;
            n += (uint32_t)__popcll(ballot(can) & 0xFFFFull);            // (costs ascend: the first candidates)
            neg[s] = 0u - 8u * (can ? w_next[s] : c_hi + 1u);
            err[s] = can ? e_next[s] : DP_INF;
        }
        ask_records(i + 1u);
        const char* row = reinterpret_cast<const char*>(rows + (size_t)(i == first ? 0u : i) * pitch);
        auto cell = [&](uint32_t at) { return reinterpret_cast<const unsigned long long*>(row + at); };
        const uint32_t here = (CHAIN_PAD + c) * 8u;
        unsigned long long v[SETS][16];
        auto addresses = [&](int s, uint32_t (&q)[4][4]) {
            row_addr_sub4<0>(here, neg[s], q[0]);
            row_addr_sub4<4>(here, neg[s], q[1]);
            row_addr_sub4<8>(here, neg[s], q[2]);
            row_addr_sub4<12>(here, neg[s], q[3]);
        };
        uint32_t polls = 0;
        auto give_up = [&]() {
            if (++polls <= ab.polls) return false;
            gave_up = true;
            if (lane == 0) atomicAdd(&ab.flags[2], 1u);
            return true;
        };
        if constexpr (SETS > 1) {
            uint32_t q[4];
            row_addr_sub4<0>(here, neg[0], q);
            while (!gave_up && ballot(cell_empty(cell_load(cell(q[0])))) != 0ull && !give_up()) asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            if (s == 0 || n > 16u * (uint32_t)s) {
                uint32_t q[4][4];
                addresses(s, q);
#pragma unroll
                for (int k = 0; k < 16; ++k) v[s][k] = __hip_atomic_load(cell(q[k >> 2][k & 3]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            } else {
#pragma unroll
                for (int k = 0; k < 16; ++k) v[s][k] = 0x7FF0000000000000ull;
            }
        }
        for (;;) {
            uint32_t top = 0u;                                           // (an empty cell has the greatest high word)
#pragma unroll
            for (int s = 0; s < SETS; ++s)
#pragma unroll
                for (int k = 0; k < 16; ++k) top = max(top, (uint32_t)(v[s][k] >> 32));
            if (ballot(top == 0xFFFFFFFFu) == 0ull || gave_up || give_up()) break;
            asm volatile("" ::: "memory");
#pragma unroll
            for (int s = 0; s < SETS; ++s) {
                if (s == 0 || n > 16u * (uint32_t)s) {
                    uint32_t q[4][4];
                    addresses(s, q);
#pragma unroll
                    for (int k = 0; k < 16; ++k)
                        if (cell_empty(v[s][k])) v[s][k] = cell_load(cell(q[k >> 2][k & 3]));
                }
            }
        }
        double t[SETS][16], best = DP_INF;
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
#pragma unroll
            for (int k = 0; k < 16; ++k) t[s][k] = __longlong_as_double((long long)v[s][k]);
            double (*t4)[4] = reinterpret_cast<double (*)[4]>(t[s]);
            acc_rec_error4<0>(t4[0], err[s], one);
            acc_rec_error4<4>(t4[1], err[s], one);
            acc_rec_error4<8>(t4[2], err[s], one);
            acc_rec_error4<12>(t4[3], err[s], one);
#pragma unroll
            for (int k = 0; k < 16; k += 4)
                best = min_f64(best, min_f64(min_f64(t[s][k], t[s][k + 1]), min_f64(t[s][k + 2], t[s][k + 3])));
        }
        cell_store(rows + (size_t)(i + 1u) * pitch + CHAIN_PAD + c, best);
        uint32_t bj = 0xFFu;
#pragma unroll
        for (int s = SETS - 1; s >= 0; --s)
#pragma unroll
            for (int k = 15; k >= 0; --k) bj = t[s][k] == best ? 16u * (uint32_t)s + (uint32_t)k : bj;
        ab.choice[(size_t)i * ab.stride + c] = (uint8_t)(best < DP_INF ? bj : 0xFFu);
        last = c <= ab.cap ? best : DP_INF;
    }
    if (halves) {
        last = wave_min_f64(last);
        if (lane == 0u) ch.least[half][c0 / 64u] = last;
    }
}

}  // namespace kimad
