// Knapsack allocation on the device (paper Appendix C; Section 3.2, Eq. optimisation).
//
// Table rows are indexed by cost in units of `unit` pairs; row i holds the least total error of
// layers 0..i at each exact cost.  Layers are visited in order, candidates in ascending j with a
// strict "<", and the answer ends at the smallest cost attaining the least total: every fp64
// add happens in the same order as in a plain sequential implementation, so the choice is
// reproducible bit for bit.
#pragma once
#include "common.h"
#include "k_compress.h"

namespace kimad {

struct AllocBuffers {
    const double* E;         // [L][J]
    const uint32_t* Ktab;    // [L][J] pairs charged for candidate j (its size, or the dense size where that is cheaper)
    const uint32_t* Kout;    // [L][J] size sent for candidate j (Ktab itself without the dense fallback)
    uint32_t L, J;
    uint64_t unit;           // cost unit in pairs
    uint32_t cap;            // capacity in units
    double* row0;            // [cap+1]
    double* row1;            // [cap+1]
    uint8_t* choice;         // [L][stride] winners (rows that fit LDS: a piece's winners of a cell side by side, k_dp_walk)
    uint16_t* cprev;         // [pieces][stride] rows that fit LDS only: the cell of the piece's first row a cell came from
    uint64_t stride;         // >= cap+1
    int32_t* j_out;
    uint64_t* K_out;
    uint64_t* offsets_out;
    int32_t* status;
    uint32_t* flags;         // [DP_FLAGS] [0] non-finite seen (rows by launch only), [1] workgroups started, [2] waits given up, [4] on: FLAG_..
    uint32_t polls;          // reads after which a wait for a row's cells is given up
    uint32_t first_ticket;   // what flags[1] starts from: 0 (a test that withholds the first workgroups: their number)
    uint32_t* info;          // [INFO_WORDS] what there is to ask of the last allocation
};

constexpr double DP_INF = __builtin_huge_val();
constexpr uint32_t DP_FLAGS = 12;
enum : uint32_t { FLAG_MET = 4u, FLAG_UNSURE = 5u, FLAG_COST = 6u, FLAG_CHAIN = 7u, FLAG_BACK = 8u, FLAG_AT_ONCE = 9u };      // (k_alloc_halves.h)
constexpr uint32_t NO_TICKET = 1u << 30;       // (no launch has so many workgroups)

// Words of AllocBuffers::info: the band's (k_alloc_band.h, 0 to 4; zero where none was run), the route taken (KIMAD_ROUTE_..) and how.
// An allocation's first kernel writes them, and what is found out later adds how.
enum : uint32_t { INFO_ROUTE = 5, INFO_HOW = 6, INFO_REPORT = 7, INFO_AHEAD = 8, INFO_STREAK = 9, INFO_WORDS = 16 };
enum : uint32_t { ROUTE_ROWS = 1, ROUTE_BAND = 2, ROUTE_TREE = 3, ROUTE_HALVES = 4 };
enum : uint32_t { HOW_ROWS = 1, HOW_FROM_LEFT = 2, HOW_AT_ONCE = 4 };     // whole rows decided; the path's totals from the left were formed; .. at once
__device__ __forceinline__ void alloc_report(const AllocBuffers& ab, uint32_t route, uint32_t thread) {
    if (thread < INFO_REPORT) ab.info[thread] = thread == INFO_ROUTE ? route : 0u;
}

// A table in which rounding may decide is often followed by others: two tensors alike make one whenever their sizes differ, and, where the
// budget covers all the others, a layer whose errors are less than some 1e-12 of the total makes one in every round.  Behind so many
// allocations in a row that whole rows had to decide, the plan's next ROWS_AHEAD go by whole rows at once, and then the tree or the halves
// are tried again.  The sizes do not hang on it.
constexpr uint32_t TIES_IN_A_ROW = 8, ROWS_AHEAD = 31;
__device__ __forceinline__ void alloc_decided(const AllocBuffers& ab, bool by_rows) {      // (one thread, where the tree or the halves have been)
    uint32_t streak = 0u;
    if (by_rows) {
        streak = min(ab.info[INFO_STREAK] + 1u, TIES_IN_A_ROW);
        if (streak == TIES_IN_A_ROW) ab.info[INFO_AHEAD] = ROWS_AHEAD;
        ab.info[INFO_HOW] = HOW_ROWS;
    }
    ab.info[INFO_STREAK] = streak;
}

// K / unit, rounded up.  (In 32 bits: a division in 64 is four times as long.)
__device__ __forceinline__ uint32_t units_of(uint32_t K, uint64_t unit) {
    if (unit >> 32) return K ? 1u : 0u;
    const uint32_t u = (uint32_t)unit, q = K / u;
    return q + (q * u != K ? 1u : 0u);
}

// Dense fallback: a layer never costs more than its bare values (n * 4 bytes), so a grid point at or beyond the
// break-even K * pair_bytes >= 4 n stands for sending the layer whole: error 0, K = n, charged
// ceil(4 n / pair_bytes) pairs (the levelling off at the uncompressed size of the paper's Section 4.2).
__global__ __launch_bounds__(256) void k_dense_view(const double* E, const uint32_t* Ktab, const LayerDesc* layers, uint32_t L,
                                                    uint32_t J, uint32_t pair_bytes, double* E_eff, uint32_t* Kcost,
                                                    uint32_t* Kout) {
    const uint32_t t = blockIdx.x * 256u + threadIdx.x;
    if (t >= L * J) return;
    const uint64_t n = layers[t / J].n, K = Ktab[t];
    const bool dense = K * pair_bytes >= n * 4ull;
    E_eff[t] = dense ? 0.0 : E[t];
    Kcost[t] = dense ? (uint32_t)((n * 4ull + pair_bytes - 1u) / pair_bytes) : (uint32_t)K;
    Kout[t] = dense ? (uint32_t)n : (uint32_t)K;
}

// Any Inf/NaN in the table?  Also seeds row 0 of the DP: 0 at cost 0, +inf elsewhere.
__global__ __launch_bounds__(256) void k_dp_init(AllocBuffers ab) {
    const uint32_t gid = blockIdx.x * 256u + threadIdx.x, gsz = gridDim.x * 256u;
    for (uint64_t t = gid; t < (uint64_t)ab.L * ab.J; t += gsz) {
        const double e = ab.E[t];
        if (!(e - e == 0.0)) atomicOr(&ab.flags[0], 1u);
    }
    for (uint64_t c = gid; c <= ab.cap; c += gsz) ab.row0[c] = c ? DP_INF : 0.0;
}

// One layer of the recurrence, one thread per cost cell (capacities too large for LDS rows).
__global__ __launch_bounds__(256) void k_dp_layer(AllocBuffers ab, uint32_t i, const double* prev, double* cur) {
    __shared__ double sE[KIMAD_MAX_J_CONST];
    __shared__ uint32_t sW[KIMAD_MAX_J_CONST];
    if (threadIdx.x < ab.J) {
        sE[threadIdx.x] = ab.E[(size_t)i * ab.J + threadIdx.x];
        sW[threadIdx.x] = units_of(ab.Ktab[(size_t)i * ab.J + threadIdx.x], ab.unit);
    }
    __syncthreads();
    const uint64_t c = (uint64_t)blockIdx.x * 256u + threadIdx.x;
    if (c > ab.cap) return;
    double best = DP_INF;
    uint32_t bj = 0xFF;
    // candidates in ascending j with a strict "<", sixteen row reads asked for at a time (a candidate that
    // costs more than the cell reads cell 0 instead and is skipped; costs ascend with j)
    constexpr int BATCH = 16;
    for (uint32_t j0 = 0; j0 < ab.J; j0 += BATCH) {
        if (sW[j0] > c) break;
        double p[BATCH];
        uint32_t w[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            w[u] = j0 + (uint32_t)u < ab.J ? sW[j0 + u] : 0xFFFFFFFFu;
            p[u] = prev[w[u] <= c ? c - w[u] : 0];
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            if (w[u] > c) continue;
            const double t = p[u] + sE[j0 + u];
            if (t < best) { best = t; bj = j0 + (uint32_t)u; }
        }
    }
    cur[c] = best;
    ab.choice[(size_t)i * ab.stride + c] = (uint8_t)bj;
}

// Candidate lists.  Candidates of one layer that cost the same number of units differ only in
// their error, and a table row is non-increasing in j: of such a run only the last (least error)
// can give the least total, and the strict "<" of the sequential scan keeps the lowest j of the
// run whose rounded total equals that least one.  So a run is evaluated at its last member and
// then backwards while the rounded total stays equal: the same winner as visiting every member, in
// about two additions instead of the run's length.  Runs whose errors are not non-increasing (only
// possible in a caller-supplied table) are kept as single candidates.  Candidates from the first
// one that costs more than the capacity are dropped (costs ascend with j).
struct DpLists {
    uint32_t* wall;  // [L][J] cost in units of candidate j
    uint32_t* w;     // [L][J] cost in units of the entry
    uint32_t* jj;    // [L][J] first member of the run | last member << 8
    double* e;       // [L][J][2] error of the last member, error of the member before it (NaN for a single)
    uint32_t* n;     // [L] entries
    uint32_t* bad;   // [L] 1 if the layer's table row holds an Inf or a NaN
    // lower convex hull of the list's (cost, error) points, for the banded recurrence
    double* he;      // [L][J] vertex errors, falling
    uint32_t* hw;    // [L][J] vertex costs, rising; HULL_LAST set at the last one
    uint32_t* hn;    // [L] vertices
    double* habs;    // [L] largest |error| of the list
};
constexpr uint32_t HULL_LAST = 0x80000000u;

// A cell of a row that nobody has stored yet (a NaN that no total can be).
constexpr unsigned long long ROW_EMPTY = ~0ull;

// Stored row r of the recurrence, `pitch` cells apart, the first `pad` of them before cost 0, by `threads` threads of which this
// is number `me`: ROW_EMPTY, and in row 0 the start.
__device__ __forceinline__ void dp_fill_row(const AllocBuffers& ab, double* rows, uint64_t pitch, uint32_t pad, uint64_t r, uint32_t me, uint32_t threads) {
    const uint64_t cells = ((uint64_t)pad + ab.cap + 64u) & ~63ull;            // (the pitch holds them)
    unsigned long long* row = reinterpret_cast<unsigned long long*>(rows + r * pitch);
    for (uint64_t x = 2ull * me; x < cells; x += 2ull * threads) {
        ulonglong2 v = make_ulonglong2(ROW_EMPTY, ROW_EMPTY);
        if (r == 0u || x < pad) v.x = x == pad ? 0ull : 0x7FF0000000000000ull;
        if (r == 0u || x + 1u < pad) v.y = 0x7FF0000000000000ull;
        *reinterpret_cast<ulonglong2*>(row + x) = v;
    }
}

// Layer i's candidate list, lane j holding candidate j: where a run starts, its last member's error and the error before it.
struct DpList {
    uint32_t w, last;              // cost in units, last member of the run that starts here
    double e, e_last, e_before;    // the candidate's own error, the last member's, that of the member before
    bool start;
    uint64_t starts, nonfinite;    // lanes where a run starts; with an Inf or a NaN
    uint64_t same;                 // members whose error is that of the one before
};
__device__ __forceinline__ DpList dp_list(const AllocBuffers& ab, uint32_t i, uint32_t j) {
    DpList d;
    const bool valid = j < ab.J;
    d.w = 0xFFFFFFFFu;
    double e = 0.0;
    if (valid) {
        d.w = units_of(ab.Ktab[(size_t)i * ab.J + j], ab.unit);
        e = ab.E[(size_t)i * ab.J + j];
    }
    d.nonfinite = ballot(valid && !(e - e == 0.0));
    const uint64_t over = ballot(valid && d.w > ab.cap);
    const uint32_t n_in = over ? (uint32_t)__builtin_ctzll(over) : ab.J;
    const uint32_t wprev = __shfl_up(d.w, 1, 64);
    const double eprev = __shfl_up(e, 1, 64);
    d.start = j < n_in && (j == 0 || d.w != wprev || !(e <= eprev));
    d.starts = ballot(d.start);
    d.e = e;
    d.same = ballot(j < n_in && !d.start && e == eprev);
    const uint64_t above = j < 63 ? d.starts & ~((2ull << j) - 1ull) : 0ull;
    d.last = (above ? (uint32_t)__builtin_ctzll(above) : n_in) - 1u;
    d.e_last = __shfl(e, (int)(d.last & 63u), 64);
    d.e_before = __shfl(e, (int)((d.last - 1u) & 63u), 64);
    return d;
}
__device__ __forceinline__ void dp_list_store(const AllocBuffers& ab, const DpLists& dl, uint32_t i, uint32_t j, const DpList& d) {
    const bool valid = j < ab.J;
    if (valid) dl.wall[(size_t)i * ab.J + j] = d.w;
    if (d.start) {
        const size_t o = (size_t)i * ab.J + (uint32_t)__builtin_popcountll(d.starts & ((1ull << j) - 1ull));
        dl.w[o] = d.w;
        dl.jj[o] = j | (d.last << 8);
        dl.e[2 * o] = d.e_last;
        dl.e[2 * o + 1] = d.last > j ? d.e_before : __longlong_as_double(0x7FF8000000000000ll);
    }
    const uint32_t n = (uint32_t)__builtin_popcountll(d.starts);
    if (valid && j >= n) dl.w[(size_t)i * ab.J + j] = 0xFFFFFFFFu;            // no entry
    if (j == 0) {
        dl.n[i] = n;
        dl.bad[i] = d.nonfinite ? 1u : 0u;
    }
}

// One wave per layer, one lane per candidate.  `with_hull`: also the list's lower convex hull.
// `rows` (not null): the stored rows of the recurrence, `pitch` cells each, the first `pad` of them before cost 0: row i + 1
// is filled with ROW_EMPTY (row 0: the start), by the gridDim.y workgroups of the layer; its counters are cleared, and `route` is reported.
// `falling` (not null): [L][J] the candidates' errors, +inf for one that is dearer than another and no better.
__global__ __launch_bounds__(64) void k_dp_prep(AllocBuffers ab, DpLists dl, uint32_t with_hull, double* rows, uint64_t pitch, uint32_t pad, double* falling,
                                                uint32_t route) {
    __shared__ double se[KIMAD_MAX_J_CONST];
    __shared__ uint32_t sw[KIMAD_MAX_J_CONST];
    const uint32_t i = blockIdx.x, j = threadIdx.x, ahead = route == ROUTE_HALVES ? ab.info[INFO_AHEAD] : 0u;
    if (rows) {
        dp_fill_row(ab, rows, pitch, pad, i + 1ull, blockIdx.y * 64u + j, 64u * gridDim.y);
        if (i == 0u) dp_fill_row(ab, rows, pitch, pad, 0ull, blockIdx.y * 64u + j, 64u * gridDim.y);
        if (i == 0u && blockIdx.y == 0u) {
            // (halves that are passed over: the chains find no number that is theirs, and leave)
            if (j < DP_FLAGS) ab.flags[j] = j == 1u ? (ahead ? NO_TICKET : ab.first_ticket) : (j == FLAG_CHAIN || j == FLAG_AT_ONCE) && ahead ? 1u : 0u;
            if (j < INFO_REPORT) ab.info[j] = j == INFO_ROUTE ? route : j == INFO_HOW && ahead ? HOW_ROWS | HOW_AT_ONCE : 0u;
            if (ahead && j == 0u) ab.info[INFO_AHEAD] = ahead - 1u;
        }
        if (blockIdx.y) return;
    }
    if (falling) {
        const double e = j < ab.J ? ab.E[(size_t)i * ab.J + j] : DP_INF;
        double least = e, largest = j < ab.J ? fabs(e) : 0.0;
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) {
            const double o = __shfl_up(least, s, 64);
            if ((int)j >= s) least = fmin(least, o);
            largest = fmax(largest, __shfl_xor(largest, s, 64));
        }
        const double before = __shfl_up(least, 1, 64);
        if (j < ab.J) falling[(size_t)i * ab.J + j] = j == 0u || e < before ? e : DP_INF;
        if (j == 0u) dl.habs[i] = largest;
    }
    const DpList d = dp_list(ab, i, j);
    dp_list_store(ab, dl, i, j, d);
    const uint32_t n = (uint32_t)__builtin_popcountll(d.starts), w = d.w;
    const uint64_t smask = d.starts;
    const bool start = d.start;
    const double e_last = d.e_last;
    if (!with_hull) return;
    // ---- the hull, one list entry per lane.  Every test below drops a point because of other points of the list
    // (one that is no dearer and saves as much; two whose chord passes at or below it), so all lanes test at once, and
    // again with their new neighbours until none is dropped.  (A point dropped or kept by the rounding of the chord test
    // changes a minimum over the vertices by rounding only.  One thread per layer pushing and popping took 17 us of the
    // next kernel; error profiles are nearly convex, and one or two rounds are the rule here.)
    const uint64_t lower = (1ull << j) - 1ull, upper = ~((2ull << j) - 1ull);
    if (start) {
        const uint32_t at = (uint32_t)__builtin_popcountll(smask & lower);
        se[at] = e_last; sw[at] = w;
    }
    __syncthreads();
    const bool listed = j < n;
    const double pe = listed ? se[j] : DP_INF;
    const uint32_t pw = listed ? sw[j] : 0xFFFFFFFFu;
    double least = pe, largest = listed ? fabs(pe) : 0.0;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const double o = __shfl_up(least, d, 64);
        if ((int)j >= d) least = fmin(least, o);
        largest = fmax(largest, __shfl_xor(largest, d, 64));
    }
    const double before = __shfl_up(least, 1, 64);
    bool alive = listed && (j == 0u || pe < before);
    uint64_t mask = ballot(alive);
    {
        const uint64_t up = mask & upper;                    // of equal costs the last, which has the least error
        const uint32_t nw = __shfl(pw, up ? __builtin_ctzll(up) : (int)j, 64);
        alive = alive && !(up && nw == pw);
        mask = ballot(alive);
    }
    for (;;) {
        const uint64_t up = mask & upper, dn = mask & lower;
        const int nx = up ? __builtin_ctzll(up) : (int)j, pv = dn ? 63 - __builtin_clzll(dn) : (int)j;
        const double ne = __shfl(pe, nx, 64), qe = __shfl(pe, pv, 64);
        const uint32_t nw = __shfl(pw, nx, 64), qw = __shfl(pw, pv, 64);
        const bool drop = alive && up && dn && (qe - pe) * (double)(nw - pw) <= (pe - ne) * (double)(pw - qw);
        const uint64_t dropped = ballot(drop);
        if (dropped == 0ull) break;
        alive = alive && !drop;
        mask &= ~dropped;
    }
    if (alive) {
        const size_t o = (size_t)i * ab.J + (uint32_t)__builtin_popcountll(mask & lower);
        dl.he[o] = pe;
        dl.hw[o] = pw | ((mask & upper) ? 0u : HULL_LAST);
    }
    if (j == 0) { dl.hn[i] = (uint32_t)__builtin_popcountll(mask); dl.habs[i] = largest; }
}

// The recurrence for capacities whose rows fit LDS, in two kernels:
//   k_dp_chain    (k_alloc_chain.h) least totals only, a min per candidate and cell, every row stored; beside that, by other
//                 workgroups of the launch, the winning candidate of every (layer, cell) pair from the stored rows;
//   k_dp_walk     one workgroup: status, smallest cost attaining the least total, back-tracking, outputs.
// Only the minimum is a sequential chain of L steps: which candidate attains it is order-independent given the previous row.
constexpr uint32_t DP_ROW_MAX = 4224;           // cells of the longest row (a discretisation factor of 4096 fits)

// min of two doubles, neither a signalling NaN (the builtin would add a canonicalising max per operand)
__device__ __forceinline__ double min_f64(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Workgroup barrier for data exchanged through LDS only.  __syncthreads() also waits for the
// acknowledgement of every global store in flight, which would put a memory round trip into each
// of the L sequential steps.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// A wave holds 16 list records per register set, record k in lane k of every 16-lane row, and
// uses them through DPP row_newbcast operands, which hand lane K of each row to all its lanes:
//   row_addr_sub4  LDS address of the row cell minus record K's cost (v_add_u32 with the negated cost)
//   acc_rec_error4 t += record K's error, as fma(error, 1.0, t): one rounding of the exact sum, the same
//                  result as an add
// Both forms were checked against a 64-lane test pattern on gfx950, four records per call.  They
// are written as inline assembly: when the compiler folds a DPP move into a subtraction itself, the instruction it emits
// applied the broadcast to the other operand in that test.  Each waits two cycles first: a DPP
// operand must not be read directly after the vector instruction that wrote it, and the compiler
// does not know that the assembly reads through DPP.
template <int K>
__device__ __forceinline__ void row_addr_sub4(uint32_t base, uint32_t neg_cost, uint32_t (&q)[4]) {
    asm("s_nop 1\n\t"
        "v_add_u32_dpp %0, %4, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_u32_dpp %1, %4, %5 row_newbcast:%7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_u32_dpp %2, %4, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_u32_dpp %3, %4, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1"
        : "=&v"(q[0]), "=&v"(q[1]), "=&v"(q[2]), "=&v"(q[3])
        : "v"(neg_cost), "v"(base), "n"(K), "n"(K + 1), "n"(K + 2), "n"(K + 3));
}
// t[u] += error of record K+u, four records at once (one wait for all of them)
template <int K>
__device__ __forceinline__ void acc_rec_error4(double (&t)[4], double err, double one) {
    asm("s_nop 1\n\t"
        "v_fmac_f64_dpp %0, %4, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f64_dpp %1, %4, %5 row_newbcast:%7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f64_dpp %2, %4, %5 row_newbcast:%8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_fmac_f64_dpp %3, %4, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf bound_ctrl:1"
        : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3])
        : "v"(err), "v"(one), "n"(K), "n"(K + 1), "n"(K + 2), "n"(K + 3));
}

// LDS pointers as 32-bit byte addresses, for address arithmetic in DPP instructions.
using lds_cdouble_ptr = const __attribute__((address_space(3))) double*;
__device__ __forceinline__ uint32_t lds_addr(const double* p) { return (uint32_t)(size_t)(lds_cdouble_ptr)p; }

// A list record as stored in LDS: x, y = the error's fp64 bits, z = minus the cost as a byte
// distance in the row.
__device__ __forceinline__ double rec_err(const uint4& r) { return __hiloint2double((int)r.y, (int)r.x); }

// The layers in pieces, whose cells k_dp_chain follows back: of four layers, and the last ones singly, since a piece's work
// begins when the chain has passed it and the last one's is waited for.  How many: more of them shorten what is waited for,
// but wait on compute units of their own, which a round's other kernels go without where the allocation runs beside them.
// (us, 12, 16, 24, 32, 40 and 48 of them.  All launches of the allocation with 64 ratios and 1001 cells, 20 layers 36.0, 31.9, 30.5,
// 30.4, 30.4, 30.5; 60 layers 55.7, 54.4, 52.2, 49.7, 46.7, 45.8; 148 layers 87.5, 86.4, 83.8, 81.9, 79.9, 77.8.  The GPT-2-shaped
// set's round with the allocation beside it 400, 400, 404, 409, 412, 415.)
struct Pieces {
    static constexpr uint32_t MOST = 4, SINGLE = 24;               // layers of a piece; last layers that are pieces
    uint32_t in_fours, fours, ones;                                // layers in pieces of four, such pieces, pieces of one
    __host__ __device__ __forceinline__ explicit Pieces(uint32_t L) {
        ones = L < SINGLE ? L : SINGLE;
        in_fours = L - ones;
        fours = (in_fours + 3u) / 4u;
    }
    __host__ __device__ __forceinline__ uint32_t count() const { return fours + ones; }
    __host__ __device__ __forceinline__ uint32_t first(uint32_t p) const {          // first layer (p = count(): the number of layers)
        return p < fours ? 4u * p : in_fours + (p - fours);
    }
    __host__ __device__ __forceinline__ uint32_t of(uint32_t layer) const {         // a layer's piece
        return layer < in_fours ? layer / 4u : fours + (layer - in_fours);
    }
};

// Status, smallest cost attaining the least total, back-tracking, outputs.  The workgroups of k_dp_chain have followed every
// cell through a piece's m layers: cprev[p][c] is the cell of piece p's first row that cell c behind its last layer came
// from, and the m winners on that way stand in bytes at choice + (first layer) stride + c m.  So the sequential part is one
// LDS read a piece; the pieces' rows are staged with one flat copy (they are contiguous, the pitch a multiple of 16 bytes),
// the first lot before the least total is known.
// `gate` (optional): a word that is zero where the allocation is already decided (k_dp_path).
constexpr uint32_t DP_STAGE_BYTES = 128u * 1024u;
constexpr uint32_t DP_WALK_MAX_L = 4224;           // layers whose path cells k_dp_walk keeps in LDS: every layer costs at least one
                                                   // cell, so a feasible path through rows of at most 4224 cells has no more layers

__global__ __launch_bounds__(1024) void k_dp_walk(AllocBuffers ab, const double* __restrict__ last, const uint32_t* __restrict__ bad,
                                                  int32_t err_infeasible, int32_t err_nonfinite, int32_t err_internal, StepLookup sl,
                                                  const uint32_t* __restrict__ gate) {
    if (gate && *gate == 0u) return;
    __shared__ __attribute__((aligned(16))) uint8_t stage[DP_STAGE_BYTES];
    __shared__ uint16_t s_cell[DP_WALK_MAX_L];     // the path's cell per piece (a store to memory in the chain would be waited for)
    __shared__ double sv[16];
    __shared__ unsigned long long sc[16];
    __shared__ uint32_t any_bad, cstar;
    __shared__ int32_t st;
    const uint32_t tid = threadIdx.x;
    const uint32_t ncell = ab.cap + 1;
    const Pieces pieces(ab.L);
    const uint32_t pitch = (uint32_t)ab.stride;                      // cells per row
    const uint32_t per_group = DP_STAGE_BYTES / (2u * pitch);
    const uint16_t* srow = reinterpret_cast<const uint16_t*>(stage);
    auto stage_rows = [&](uint32_t lo_p, uint32_t nrows) {
        const uint4* from = reinterpret_cast<const uint4*>(ab.cprev + (size_t)lo_p * pitch);
        uint4* dst = reinterpret_cast<uint4*>(stage);
        const uint32_t n16 = nrows * (pitch / 8u);
        for (uint32_t x0 = 0; x0 < n16; x0 += 8u * 1024u) {
            uint4 v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t x = x0 + k * 1024u + tid;
                v[k] = x < n16 ? from[x] : make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t x = x0 + k * 1024u + tid;
                if (x < n16) dst[x] = v[k];
            }
        }
    };
    if (tid == 0) any_bad = 0u;
    __syncthreads();
    uint32_t mybad = 0;
    for (uint32_t i = tid; i < ab.L; i += 1024) mybad |= bad[i];
    if (mybad) atomicOr(&any_bad, 1u);
    // least total, smallest cost attaining it
    double best = DP_INF;
    uint32_t bc = 0xFFFFFFFFu;
    for (uint32_t c = tid; c < ncell; c += 1024) {
        const double v = last[c];
        if (v < best) { best = v; bc = c; }
    }
    uint32_t hi = pieces.count(), lo_p = hi > per_group ? hi - per_group : 0u;
    if (ab.L <= DP_WALK_MAX_L) stage_rows(lo_p, hi - lo_p);
    auto least = [&](int d) {
        const double ov = __shfl_xor(best, d, 64);
        const uint32_t oc = __shfl_xor(bc, d, 64);
        if (ov < best || (ov == best && oc < bc)) { best = ov; bc = oc; }
    };
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) least(d);
    if (lane_id() == 0) { sv[tid >> 6] = best; sc[tid >> 6] = bc; }
    __syncthreads();
    if (tid < 64u) {
        best = sv[tid & 15u];
        bc = (uint32_t)sc[tid & 15u];
#pragma unroll
        for (int d = 8; d > 0; d >>= 1) least(d);
        if (tid == 0) {
            int32_t s = 0;
            if (any_bad) s = err_nonfinite;
            else if (ab.flags[2]) s = err_internal;
            else if (!(best < DP_INF) || ab.L > DP_WALK_MAX_L) s = err_infeasible;   // (more layers than cells: no finite total)
            st = s;
            cstar = bc;
            *ab.status = s;
        }
    }
    __syncthreads();
    if (st != 0) {
        for (uint32_t i = tid; i < ab.L; i += 1024) { ab.j_out[i] = 0; ab.K_out[i] = 0; }
        for (uint32_t i = tid; i <= ab.L; i += 1024) ab.offsets_out[i] = 0;
        step_lookup(sl, 1024u);
        return;
    }
    for (;;) {
        if (tid == 0) {
            uint32_t c = cstar;
            for (uint32_t p = hi; p-- > lo_p;) {
                s_cell[p] = (uint16_t)c;
                c = min((uint32_t)srow[(size_t)(p - lo_p) * pitch + c], ab.cap);
            }
            cstar = c;
        }
        hi = lo_p;
        __syncthreads();
        if (hi == 0u) break;
        lo_p = hi > per_group ? hi - per_group : 0u;
        stage_rows(lo_p, hi - lo_p);
        __syncthreads();
    }
    // winners along the path, sizes and offsets, in parallel
    unsigned long long carry = 0;
    for (uint32_t i0b = 0; i0b < ab.L; i0b += 1024) {
        const uint32_t i = i0b + tid;
        unsigned long long K = 0;
        if (i < ab.L) {
            const uint32_t p = pieces.of(i), first = pieces.first(p), m = pieces.first(p + 1u) - first;
            const uint32_t j = ab.choice[(size_t)first * ab.stride + (size_t)s_cell[p] * m + (i - first)];
            ab.j_out[i] = (int32_t)j;
            K = ab.Kout[(size_t)i * ab.J + j];
            ab.K_out[i] = K;
        }
        unsigned long long tot;
        const unsigned long long ex = block_exclusive_scan<unsigned long long>(K, sc, &tot);
        if (i < ab.L) ab.offsets_out[i] = carry + ex;
        carry += tot;
    }
    if (tid == 0) ab.offsets_out[ab.L] = carry;
    step_lookup(sl, 1024u);
}

// Smallest cost attaining the least total, back-tracking, outputs.  One workgroup.
// `bad` (not null): per layer, whether its table row holds an Inf or a NaN; else flags[0] says it of the table.
// `gate`: as in k_dp_walk.
__global__ __launch_bounds__(1024) void k_dp_final(AllocBuffers ab, const double* last, const uint32_t* __restrict__ bad,
                                                   int32_t err_infeasible, int32_t err_nonfinite, int32_t err_internal, StepLookup sl,
                                                   const uint32_t* __restrict__ gate) {
    if (gate && *gate == 0u) return;
    __shared__ double sv[16];
    __shared__ unsigned long long sc[16];
    __shared__ unsigned long long cstar;
    __shared__ uint32_t any_bad;
    __shared__ int32_t st;
    const uint32_t tid = threadIdx.x;
    if (tid == 0) any_bad = bad ? 0u : ab.flags[0];
    if (!bad) alloc_report(ab, ROUTE_ROWS, tid);           // (no kernel of a launch per layer has)
    __syncthreads();
    if (bad) {
        uint32_t mine = 0u;
        for (uint32_t i = tid; i < ab.L; i += 1024u) mine |= bad[i];
        if (mine) atomicOr(&any_bad, 1u);
    }
    double best = DP_INF;
    unsigned long long bc = ~0ull;
    for (uint64_t c0 = tid; c0 <= ab.cap; c0 += 8u * 1024u) {
        double v[8];                            // eight loads at a time (positions past the end read the last cell and are dropped)
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = last[min(c0 + 1024u * (uint64_t)u, (uint64_t)ab.cap)];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint64_t c = c0 + 1024u * (uint64_t)u;
            if (c <= ab.cap && v[u] < best) { best = v[u]; bc = c; }     // ascending c per thread: keeps the smallest
        }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const double ov = __shfl_xor(best, d, 64);
        const unsigned long long oc = __shfl_xor(bc, d, 64);
        if (ov < best || (ov == best && oc < bc)) { best = ov; bc = oc; }
    }
    if (lane_id() == 0) { sv[tid >> 6] = best; sc[tid >> 6] = bc; }
    __syncthreads();
    if (tid == 0) {
        for (uint32_t w = 1; w < 16; ++w)
            if (sv[w] < best || (sv[w] == best && sc[w] < bc)) { best = sv[w]; bc = sc[w]; }
        int32_t s = 0;
        if (any_bad) s = err_nonfinite;
        else if (bad && ab.flags[2]) s = err_internal;
        else if (!(best < DP_INF)) s = err_infeasible;
        st = s;
        cstar = bc;
        *ab.status = s;
    }
    __syncthreads();
    if (st != 0) {
        for (uint32_t i = tid; i < ab.L; i += 1024) { ab.j_out[i] = 0; ab.K_out[i] = 0; }
        for (uint32_t i = tid; i <= ab.L; i += 1024) ab.offsets_out[i] = 0;
        step_lookup(sl, 1024u);
        return;
    }
    // Back-tracking, two layers per memory round trip: with the cell's own choice, lane j asks for the layer before's
    // choice at the cell that candidate j would lead to; the lane that the choice names has the next one.  The
    // candidates' costs wait in LDS (when the table fits) so that the chain holds no second memory read
    // and no division; sizes and offsets follow in parallel.  (One choice per round trip, by one thread, and one load at
    // a time above: 44 us for 58 layers and 58 thousand cells, 34 now.)
    constexpr uint32_t W_LDS = 12288;
    __shared__ uint32_t sw[W_LDS];
    const uint32_t LJ = ab.L * ab.J;
    const bool w_in_lds = LJ <= W_LDS;
    if (w_in_lds)
        for (uint32_t t = tid; t < LJ; t += 1024) sw[t] = units_of(ab.Ktab[t], ab.unit);
    __syncthreads();
    if (tid < 64) {
        static_assert(KIMAD_MAX_J_CONST <= 64, "one lane per candidate");
        uint64_t c = cstar;
        const uint32_t j = min(tid, ab.J - 1u);
        auto cost = [&](uint32_t i, uint32_t k) { return w_in_lds ? sw[i * ab.J + k] : units_of(ab.Ktab[(size_t)i * ab.J + k], ab.unit); };
        for (uint32_t i = ab.L; i > 0u;) {
            --i;
            const uint32_t w = cost(i, j);
            const uint32_t here = ab.choice[(size_t)i * ab.stride + c];
            uint32_t before = 0u;
            if (i > 0u) before = ab.choice[(size_t)(i - 1u) * ab.stride + (w <= c ? c - w : 0u)];
            const int j0 = (int)__builtin_amdgcn_readfirstlane(here);          // (a feasible path meets candidates only)
            if (tid == 0) ab.j_out[i] = j0;
            c -= (uint32_t)__builtin_amdgcn_readlane((int)w, j0);
            if (i == 0u) break;
            --i;
            const uint32_t j1 = (uint32_t)__builtin_amdgcn_readlane((int)before, j0);
            if (tid == 0) ab.j_out[i] = (int32_t)j1;
            c -= cost(i, j1);
        }
    }
    __threadfence_block();
    __syncthreads();
    unsigned long long carry = 0;
    for (uint32_t i0b = 0; i0b < ab.L; i0b += 1024) {
        const uint32_t i = i0b + tid;
        unsigned long long K = 0;
        if (i < ab.L) {
            K = ab.Kout[(size_t)i * ab.J + (uint32_t)ab.j_out[i]];
            ab.K_out[i] = K;
        }
        unsigned long long tot;
        const unsigned long long ex = block_exclusive_scan<unsigned long long>(K, sc, &tot);
        if (i < ab.L) ab.offsets_out[i] = carry + ex;
        carry += tot;
    }
    if (tid == 0) ab.offsets_out[ab.L] = carry;
    step_lookup(sl, 1024u);
}

}  // namespace kimad
