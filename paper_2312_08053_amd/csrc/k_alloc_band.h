// Knapsack allocation inside a band of cost cells (paper Appendix C; Section 3.2, Eq. optimisation).
//
// The recurrence of k_alloc.h visits every cost cell of every layer although the least total runs
// through a narrow corridor of them.  Two kernels cut the work down to that corridor without
// changing one bit of the result:
//
//   k_dp_bounds  Lagrangian bounds.  For a multiplier lambda >= 0 and any assignment,
//                    sum_i E_i  >=  sum_i min_k (E_ik + lambda w_ik)  -  lambda * (sum_i w_i),
//                so a path through cell c of row r (layers 0..r-1 spent exactly c units) totals at least
//                    max_lambda [A_r(lambda) - lambda c]  +  max_lambda [B_r(lambda) - lambda (cap - c)],
//                A_r, B_r the sums of the per-layer minima over the layers before / from r.  Any feasible
//                assignment gives an upper bound UB on the least total.  A cell whose lower bound exceeds
//                UB (by a margin far above the rounding of these sums) lies on no path that attains the
//                least total, and the cells that remain form an interval of every row: its band.
//   k_dp_banded  the recurrence on the band cells only; sources outside the previous row's band count
//                as +inf.  Then the walk back and the outputs.
//
// Why the result is the same.  The sequential recurrence computes, per cell, the minimum over paths of
// the path's left-to-right fp64 sum, and fp64 addition is monotone, so removing cells can only raise
// a cell's value.  Every cell of a path that attains the least total T stays in its band (its lower
// bound is at most the path's real sum <= T (1 + tiny) <= UB (1 + tiny)); by induction along such a path
// each of its cells keeps its value and its winning candidate: the first candidate, in list order,
// that attains the cell's minimum comes from a cell that is itself on such a path, so it is in the
// band with its value unchanged, and the candidates before it still do not attain the minimum.  The
// last row therefore has the same minimum at the same cells, and back-tracking meets unchanged cells only.
#pragma once
#include "common.h"
#include "k_alloc.h"
#include "k_alloc_chain.h"

namespace kimad {

constexpr uint32_t BAND_MAX_L = 1024;          // layers the banded allocation handles
constexpr uint32_t BAND_LCAP = 7168;           // list records (and so hull vertices, which LDS holds) the bounds kernel takes
constexpr uint32_t BAND_NLAM = 32;             // multipliers around the one found: lambda* rho^(m - 16)
constexpr uint32_t BAND_GREEDY = 16;           // rounds of the greedy fill that tightens the upper bound
constexpr uint32_t BOUNDS_THREADS = 1024;
constexpr uint32_t BAND_EDGES_PER_THREAD = BAND_LCAP / BOUNDS_THREADS;   // 7
constexpr uint32_t BAND_GROUPS = BOUNDS_THREADS / BAND_NLAM;             // 32 groups of layers, one thread per multiplier each

struct BandBuffers {
    uint32_t* lo;          // [L + 1] first cell of row r's band (row 0 is the start: cell 0)
    uint32_t* hi;          // [L + 1] last cell
    uint32_t* info;        // [INFO_WORDS] max width, sum of widths, 1 if the bands are the whole rows, upgrades taken, 1 if nothing fits
    // the list records that can connect the bands of rows i and i + 1 (the only ones the banded recurrence visits)
    uint32_t* live;        // [L] first record | count << 8
    double* table;         // [(L + 1) * BAND_NLAM] prefix sums of the per-layer minima; the rows' memory before there are rows
};

__device__ __forceinline__ double max_f64(double a, double b) {   // neither a signalling NaN (see min_f64)
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// maximum over the T lanes of a group (T = 1, 2, 4, 8), in every lane of it
template <int T>
__device__ __forceinline__ double group_max(double v) {
    if (T >= 2) v = max_f64(v, dpp_f64<0xB1>(v));      // quad_perm [1,0,3,2]
    if (T >= 4) v = max_f64(v, dpp_f64<0x4E>(v));      // quad_perm [2,3,0,1]
    if (T >= 8) v = max_f64(v, dpp_f64<0x141>(v));     // row_half_mirror: the other quad of the eight
    return v;
}

// The greedy fill, by one wave: lane l looks after layers l, l + 64, ...  Every round the steepest edge that fits what is
// left is taken (the lowest lane's among equals; only the upper bound's tightness depends on it); returns the steps taken.
// Up to 64 M layers' next edges stay in registers; beyond (M = 0) they are read again every round.  (One thread per layer
// of the whole workgroup, with two barriers a round, took 20 us.)
template <int M>
__device__ __forceinline__ uint32_t greedy_fill(const double* HE, const uint32_t* HW, const uint16_t* s_off, uint16_t* s_q,
                                                uint32_t L, uint32_t left) {
    constexpr int R = M ? M : 1;
    const uint32_t lane = lane_id();
    double slope[R];
    uint32_t dw[R];
    auto edge = [&](uint32_t i, double& s, uint32_t& d) {
        const uint32_t o = (uint32_t)s_off[i] + s_q[i];
        const uint32_t w = HW[o];
        s = 0.0; d = 0xFFFFFFFFu;
        if (!(w & HULL_LAST)) {
            d = (HW[o + 1u] & ~HULL_LAST) - w;
            s = (HE[o] - HE[o + 1u]) / (double)d;
        }
    };
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const uint32_t i = lane + 64u * (uint32_t)m;
        slope[m] = 0.0; dw[m] = 0xFFFFFFFFu;
        if (i < L) edge(i, slope[m], dw[m]);
    }
    uint32_t taken = 0u;
    for (uint32_t round = 0; round < BAND_GREEDY && left > 0u; ++round) {
        double best = 0.0;
        uint32_t which = 0u, cost = 0u;
        if (M) {
#pragma unroll
            for (int m = 0; m < M; ++m)
                if (dw[m] <= left && slope[m] > best) { best = slope[m]; which = (uint32_t)m; cost = dw[m]; }
        } else {
            for (uint32_t i = lane; i < L; i += 64u) {
                double s;
                uint32_t d;
                edge(i, s, d);
                if (d <= left && s > best) { best = s; which = i / 64u; cost = d; }
            }
        }
        double top = best;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) top = max_f64(top, __shfl_xor(top, d, 64));
        if (!(top > 0.0)) break;
        const uint32_t winner = (uint32_t)__builtin_ctzll(ballot(best == top));
        left -= (uint32_t)__builtin_amdgcn_readlane((int)cost, (int)winner);
        ++taken;
        if (lane == winner) {
            const uint32_t i = lane + 64u * which;
            s_q[i] = (uint16_t)(s_q[i] + 1u);
            double s = 0.0;
            uint32_t d = 0u;
            if (M) edge(i, s, d);
#pragma unroll
            for (int m = 0; m < M; ++m)
                if (which == (uint32_t)m) { slope[m] = s; dw[m] = d; }
        }
        wave_sync_lds();
    }
    return taken;
}

// Bounds kernel: one workgroup of sixteen waves over the hulls of k_dp_prep.  Only hull vertices can minimise E + lambda w,
// and along a hull the slopes (error saved per unit of cost) fall, so a layer's minimiser for a given lambda is found by
// bisection.
//   1  the hulls go to LDS;
//   2  the smallest lambda whose minimisers fit the capacity: the total cost at lambda is that of the cheapest
//      vertices plus the cost steps of all hull edges steeper than lambda; every thread keeps a few edges in
//      registers and the bit pattern of lambda (ordered like the doubles) is searched;
//   3  upper bound: that assignment, then up to BAND_GREEDY single steps to a next hull vertex;
//   4  the table A[r][m] = sum over layers before r of the minimum at lambda_m: a thread per multiplier and group of
//      consecutive layers sums its layers, the groups' totals are added up afterwards;
//   5  the band of every row by a search outward from the assignment's own cell, four threads to an edge;
//   6  the live records of every layer.
// A chain of short phases, each a few LDS round trips: 92 us with the hulls, serial sums and the live records' copies in
// it, 47 us now on the headline set's table at 4097 cells (148 layers).
__global__ __launch_bounds__(BOUNDS_THREADS) void k_dp_bounds(AllocBuffers ab, DpLists dl, BandBuffers bb) {
    constexpr uint32_t NWAVES = BOUNDS_THREADS / 64;
    __shared__ double HE[BAND_LCAP];                                    // 56 KB: vertex errors
    __shared__ uint32_t HW[BAND_LCAP];                                  // 28 KB: vertex costs, HULL_LAST at a hull's last
    __shared__ double s_gt[BAND_GROUPS * BAND_NLAM];                    // 8 KB: per group and multiplier, then the sums before the group
    __shared__ uint16_t s_off[BAND_MAX_L], s_hn[BAND_MAX_L], s_q[BAND_MAX_L], s_n[BAND_MAX_L];
    __shared__ uint16_t s_cum[BAND_MAX_L + 2], s_blo[BAND_MAX_L + 2], s_bhi[BAND_MAX_L + 2];
    __shared__ uint32_t su[16];
    __shared__ double sd[16];
    __shared__ double s_lam[BAND_NLAM], s_btot[BAND_NLAM];
    __shared__ uint32_t s_hist[2][64];
    __shared__ uint32_t s_flag, s_wmax, s_upgrades;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t L = ab.L, J = ab.J, cap = ab.cap;

    if (tid == INFO_ROUTE || tid == INFO_HOW) bb.info[tid] = tid == INFO_ROUTE ? ROUTE_BAND : 0u;
    // no bound to use: whole rows, every record live (or, if `hopeless`, nothing fits and the recurrence is not run)
    auto whole_rows = [&](bool hopeless) {
        for (uint32_t r = tid; r <= L; r += BOUNDS_THREADS) { bb.lo[r] = 0u; bb.hi[r] = r ? cap : 0u; }
        if (tid < L) bb.live[tid] = min(dl.n[tid], 64u) << 8;
        if (tid == 0) { bb.info[0] = cap + 1u; bb.info[1] = L * (cap + 1u); bb.info[2] = 1u; bb.info[3] = 0u; bb.info[4] = hopeless ? 1u : 0u; }
    };

    // ---- 1: sizes, offsets, hulls into LDS
    const uint32_t my_n = tid < L ? min(dl.hn[tid], 64u) : 0u;
    const uint32_t list_n = tid < L ? min(dl.n[tid], 64u) : 0u;
    const double my_abs = tid < L ? dl.habs[tid] : 0.0;
    const uint32_t my_bad = tid < L ? dl.bad[tid] : 0u;
    uint32_t n_tot, list_tot;
    const uint32_t my_off = block_exclusive_scan<uint32_t>(my_n, su, &n_tot);
    (void)block_exclusive_scan<uint32_t>(list_n, su, &list_tot);
    if (tid == 0) { s_flag = 0u; s_wmax = 0u; s_upgrades = 0u; }
    if (tid < 128u) s_hist[tid >> 6][tid & 63u] = 0u;
    if (tid < L && list_tot <= BAND_LCAP) { s_hn[tid] = (uint16_t)my_n; s_n[tid] = (uint16_t)list_n; s_off[tid] = (uint16_t)my_off; }
    __syncthreads();
    if (my_bad) atomicOr(&s_flag, 1u);
    if (tid < L && my_n == 0u) atomicOr(&s_flag, 2u);                    // a layer with no affordable candidate
    __syncthreads();
    if (list_tot > BAND_LCAP || s_flag != 0u) { whole_rows((s_flag & 2u) != 0u); return; }
    // eight layers' loads in flight per wave
    for (uint32_t i0 = wave * 8u; i0 < L; i0 += NWAVES * 8u) {
        double e[8];
        uint32_t w[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t i = i0 + (uint32_t)u;
            const bool in = i < L && lane < s_hn[min(i, L - 1u)];
            const size_t o = in ? (size_t)i * J + lane : 0;
            e[u] = dl.he[o]; w[u] = dl.hw[o];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t i = i0 + (uint32_t)u;
            if (i < L && lane < s_hn[i]) { HE[s_off[i] + lane] = e[u]; HW[s_off[i] + lane] = w[u]; }
        }
    }
    __syncthreads();
    auto cost_at = [&](uint32_t o) { return HW[o] & ~HULL_LAST; };
    // the vertex of layer i that minimises E + lam w: the number of its edges steeper than lam
    auto vertex_at = [&](uint32_t i, double lam) {
        const uint32_t o = s_off[i];
        uint32_t lo = 0u, hi = (uint32_t)s_hn[i] - 1u;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (HE[o + mid] - HE[o + mid + 1u] > lam * (double)(cost_at(o + mid + 1u) - HW[o + mid])) lo = mid + 1u; else hi = mid;
        }
        return lo;
    };

    // ---- 2: the smallest multiplier that fits.  This thread's edges (slope, cost step) stay in registers.
    unsigned long long lo_b = 0ull, hi_b = 0ull;
    double gentle;                                                           // the least steep edge
    {
        double sl[BAND_EDGES_PER_THREAD];
        uint32_t dw[BAND_EDGES_PER_THREAD];
        double steep = 0.0;
        gentle = DP_INF;
#pragma unroll
        for (int u = 0; u < (int)BAND_EDGES_PER_THREAD; ++u) {
            const uint32_t x = tid + (uint32_t)u * BOUNDS_THREADS;
            sl[u] = 0.0; dw[u] = 0u;
            if (x < n_tot && !(HW[x] & HULL_LAST)) {
                dw[u] = cost_at(x + 1u) - HW[x];
                sl[u] = (HE[x] - HE[x + 1u]) / (double)dw[u];
                steep = max_f64(steep, sl[u]);
                gentle = min_f64(gentle, sl[u]);
            }
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) { steep = max_f64(steep, __shfl_xor(steep, d, 64)); gentle = min_f64(gentle, __shfl_xor(gentle, d, 64)); }
        if (lane == 0) { sd[wave] = steep; s_lam[wave] = gentle; }
        uint32_t cheapest;
        (void)block_exclusive_scan<uint32_t>(tid < L ? cost_at(my_off) : 0u, su, &cheapest);        // (has barriers)
        for (uint32_t v = 0; v < NWAVES; ++v) { steep = max_f64(steep, sd[v]); gentle = min_f64(gentle, s_lam[v]); }
        __syncthreads();
        if (cheapest > cap) { whole_rows(true); return; }                    // nothing fits
        const uint32_t room = cap - cheapest;
        // The smallest multiplier (as a bit pattern: non-negative doubles order like their patterns) at which the
        // edges steeper than it fit the room.  Sixty-four-way search: the patterns between lo_b (does not fit, or 0)
        // and lo_b + 2^k are cut into 64 buckets, every edge inside adds its cost step to its bucket in LDS, and
        // every wave finds for itself the lowest bucket boundary at which what lies above fits: six bits of the
        // pattern per round and two barriers, down to a gap of 2^27 patterns (2^-25 relative: closer breakpoints
        // make no difference worth a round).
        uint32_t above = 0u;                                                 // cost steps of the edges at or beyond lo_b + 2^k
        uint32_t buf = 0u;
        for (int k = 63; k > 27; k -= 6) {
            const int sh = k - 6;                                            // log2 of a bucket's size
#pragma unroll
            for (int u = 0; u < (int)BAND_EDGES_PER_THREAD; ++u) {
                const unsigned long long bits = (unsigned long long)__double_as_longlong(sl[u]);
                // bucket b holds the patterns in (lo_b + b 2^sh, lo_b + (b + 1) 2^sh]
                if (dw[u] && bits > lo_b && ((bits - lo_b - 1ull) >> sh) < 64ull)
                    atomicAdd(&s_hist[buf][(uint32_t)((bits - lo_b - 1ull) >> sh)], dw[u]);
            }
            __syncthreads();
            const uint32_t mine = s_hist[buf][lane];
            s_hist[buf ^ 1u][lane] = 0u;                                     // the other table, for the next round
            const uint32_t inc = wave_scan_add_u32(mine);                    // buckets 0..lane
            const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
            const uint32_t from_here = tot - inc + mine;                     // buckets lane..63
            // cost at boundary m (edges strictly above lo_b + m 2^sh) = above + buckets m..63
            const uint64_t fits = ballot(above + from_here <= room);
            // boundary 64 always fits (the invariant); the lowest fitting boundary of 0..63, if any
            const uint32_t m = fits ? (uint32_t)__ffsll((long long)fits) - 1u : 64u;
            const uint32_t keep = m < 64u ? (uint32_t)__builtin_amdgcn_readlane((int)from_here, (int)min(m, 63u)) : 0u;
            above += keep;
            hi_b = lo_b + ((unsigned long long)m << sh);
            if (m > 0u) lo_b += (unsigned long long)(m - 1u) << sh;          // boundary m - 1 does not fit
            __syncthreads();
            buf ^= 1u;
            if (m == 0u) {
                // boundary 0 itself fits: either everything fits (lo_b = 0: the multiplier is 0) or the gap has
                // closed onto a pattern that does not fit and its successor that does
                break;
            }
            // the next round looks inside (boundary m - 1, boundary m], a range of 2^sh patterns
        }
        // (a first round that finds even its last boundary too low ends beyond the finite patterns: the steepest
        // slope itself always fits, nothing being steeper)
        hi_b = min(hi_b, (unsigned long long)__double_as_longlong(steep));
    }
    // (a little above, so that an edge as steep as the multiplier is not taken by the rounding of vertex_at's product)
    const double lam_star = __longlong_as_double((long long)hi_b) * (1.0 + 1e-12);

    // ---- 3: a feasible assignment and its total
    if (tid < L) s_q[tid] = (uint16_t)vertex_at(tid, lam_star);
    uint32_t used;
    (void)block_exclusive_scan<uint32_t>(tid < L ? cost_at(my_off + s_q[tid]) : 0u, su, &used);      // (its own s_q: no barrier needed before)
    if (used > cap) { whole_rows(false); return; }                            // (cannot happen; a bound that is no bound must not be used)
    if (wave == 0u) {
        const uint32_t taken = L <= 256u ? greedy_fill<4>(HE, HW, s_off, s_q, L, cap - used) : greedy_fill<0>(HE, HW, s_off, s_q, L, cap - used);
        if (lane == 0) s_upgrades = taken;
    }
    __syncthreads();
    double ub, abs_tot;
    (void)block_exclusive_scan<double>(tid < L ? HE[my_off + s_q[tid]] : 0.0, sd, &ub);
    (void)block_exclusive_scan<double>(my_abs, sd, &abs_tot);
    {
        const uint32_t w_mine = tid < L ? cost_at(my_off + s_q[tid]) : 0u;
        const uint32_t before = block_exclusive_scan<uint32_t>(w_mine, su, nullptr);
        if (tid < L) s_cum[tid + 1u] = (uint16_t)(before + w_mine);
        if (tid == 0) s_cum[0] = 0u;
    }
    const double ub_m = ub + 1e-9 * (fabs(ub) + abs_tot);
    // Errors times costs must stay inside the doubles (a hull test whose products overflow drops true vertices, and the bound
    // is none), and the margin above the smallest denormal times the layers.
    if (!(abs_tot <= 1e290) || (abs_tot > 0.0 && abs_tot < 1e-290)) { whole_rows(false); return; }
    if (!(gentle <= 1e300)) gentle = 0.0;                                     // one vertex per layer

    // ---- 4: multipliers around lam_star (around the least steep slope if everything fits); per (layer, multiplier) the
    // minimum, summed over the layers
    if (tid < BAND_NLAM) {
        const double base = lam_star > 0.0 ? lam_star : gentle;
        double f = 1.0;
        const int p = (int)tid - (int)(BAND_NLAM / 2u);
        for (int q = 0; q < (p < 0 ? -p : p); ++q) f *= 1.15;
        s_lam[tid] = p < 0 ? base / f : base * f;
    }
    __syncthreads();
    const uint32_t m_mine = tid % BAND_NLAM, g_mine = tid / BAND_NLAM, per_group = (L + BAND_GROUPS - 1u) / BAND_GROUPS;
    {
        const double lam = s_lam[m_mine];
        double run = 0.0;
        const uint32_t i1 = min(L, (g_mine + 1u) * per_group);
        for (uint32_t i = g_mine * per_group; i < i1; ++i) {
            const uint32_t o = s_off[i] + vertex_at(i, lam);
            run += HE[o] + lam * (double)cost_at(o);
            bb.table[(size_t)(i + 1u) * BAND_NLAM + m_mine] = run;
        }
        s_gt[tid] = run;
    }
    __syncthreads();
    {
        double before = 0.0;
        for (uint32_t g = 0; g < g_mine; ++g) before += s_gt[g * BAND_NLAM + m_mine];
        const double mine = s_gt[tid];
        __syncthreads();
        s_gt[tid] = before;
        if (g_mine == BAND_GROUPS - 1u) s_btot[m_mine] = before + mine;
    }
    __syncthreads();

    // ---- 5: the band of every row: four threads an edge, eight multipliers each, towards cell 0 and towards the last
    for (uint32_t x0 = 0u; x0 < 2u * L; x0 += BOUNDS_THREADS / 4u) {
        constexpr int T = 4, PT = (int)BAND_NLAM / T;
        const uint32_t x = x0 + tid / T, part = tid % T, side = x & 1u;
        const bool mine = x < 2u * L;
        const uint32_t r = mine ? (x >> 1) + 1u : L;                          // (lanes past the last row repeat it: a group's lanes stay together)
        double a[PT], lm[PT], bt[PT];
#pragma unroll
        for (int u = 0; u < PT; ++u) {
            const uint32_t m = part + (uint32_t)u * T;
            a[u] = bb.table[(size_t)r * BAND_NLAM + m] + s_gt[(r - 1u) / per_group * BAND_NLAM + m];
            lm[u] = s_lam[m]; bt[u] = s_btot[m] - a[u];
        }
        auto within = [&](uint32_t c) {
            const double cd = (double)c, rd = (double)(cap - c);
            double pre = a[0] - lm[0] * cd, suf = bt[0] - lm[0] * rd;
#pragma unroll
            for (int u = 1; u < PT; ++u) {
                pre = max_f64(pre, a[u] - lm[u] * cd);
                suf = max_f64(suf, bt[u] - lm[u] * rd);
            }
            return group_max<T>(pre) + group_max<T>(suf) <= ub_m;
        };
        // Steps of 8, 32, 128, ... away from the assignment's own cell until a probe falls outside (or the row's end is
        // inside), then bisection between the last cell inside and the first outside.
        const uint32_t on_path = s_cum[r];
        const uint32_t room = side ? cap - on_path : on_path;                // cells between the path and the row's end
        uint32_t in = 0u, out = room + 1u, stepd = 8u;                       // distances from the path: `in` inside, `out` outside (room + 1: beyond the row)
        while (out - in > 1u) {
            uint32_t probe;
            if (out == room + 1u) { probe = min(in + stepd, room); stepd *= 4u; }
            else probe = in + (out - in) / 2u;
            if (within(side ? on_path + probe : on_path - probe)) { in = probe; if (probe == room) break; }
            else out = probe;
        }
        if (mine && part == 0u) {
            const uint32_t edge = side ? on_path + in : on_path - in;
            if (side) { bb.hi[r] = edge; s_bhi[r] = (uint16_t)edge; } else { bb.lo[r] = edge; s_blo[r] = (uint16_t)edge; }
        }
    }
    if (tid == 0) { bb.lo[0] = 0u; bb.hi[0] = 0u; s_blo[0] = 0u; s_bhi[0] = 0u; }
    __syncthreads();

    // ---- 6: the records that can connect the bands of rows i and i + 1: a cell of each differ by a cost in
    // [lo' - hi, hi' - lo]; costs ascend along a list, so they are a run of it
    for (uint32_t i0 = wave * 8u; i0 < L; i0 += NWAVES * 8u) {
        uint32_t w[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t i = min(i0 + (uint32_t)u, L - 1u);
            w[u] = dl.w[(size_t)i * J + min(lane, (uint32_t)s_n[i] - 1u)];   // (every list has an entry)
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t i = i0 + (uint32_t)u;
            if (i >= L) break;
            const uint32_t plo = s_blo[i], phi = s_bhi[i], clo = s_blo[i + 1u], chi = s_bhi[i + 1u];
            const uint32_t w_min = clo > phi ? clo - phi : 0u;
            const uint64_t in = ballot(lane < s_n[i] && w[u] >= w_min && w[u] + plo <= chi);
            if (lane == 0) bb.live[i] = in ? (uint32_t)__builtin_ctzll(in) | ((uint32_t)__popcll(in) << 8) : 0u;
        }
    }
    // diagnostics
    const uint32_t width = tid < L ? (uint32_t)s_bhi[tid + 1u] - (uint32_t)s_blo[tid + 1u] + 1u : 0u;
    uint32_t wsum;
    (void)block_exclusive_scan<uint32_t>(width, su, &wsum);
    if (width) atomicMax(&s_wmax, width);
    __syncthreads();
    if (tid == 0) { bb.info[0] = s_wmax; bb.info[1] = wsum; bb.info[2] = 0u; bb.info[3] = s_upgrades; bb.info[4] = 0u; }
}

// The recurrence on the band cells, by one workgroup, then the walk back and the outputs.
//
// The chain of L layers is sequential and a layer is little work (tens to hundreds of cells, a few records each), so what
// counts is the length of one layer's dependent steps: a barrier, one LDS read of the previous row, an addition and a
// minimum.  The layer loop therefore computes values only, in LDS, indexed from the band's first cell: a wave looks after
// sixteen cells, the same ones in each of its four 16-lane rows, lane 16 r + k holds live record 4 k + r and hands it to
// its row by DPP, and a minimum over the rows closes the layer (as in k_dp_chain); which record attained it is asked along
// the optimal path alone, afterwards.  A row ends with a cell of +inf, which sources outside the band read.  Only the
// records that can connect the bands are visited; they wait in LDS, a group of layers at a time, and a layer's are read
// one layer ahead.
//
// All rows stay in LDS if they fit (BAND_CELLS), else two of them do and every row is also written to memory, from where
// the walk stages them again, as many layers at a time as fit.
//
// The walk: at a layer and cell, lane k tests record k: the first, in list order, whose total equals the cell's value
// is the one the sequential scan with a strict "<" would have kept.  One wave, two LDS reads deep per layer.  The lowest
// member of a winner's run with the same rounded total, sizes and offsets follow for all layers in parallel.
//
// As many waves stay for the layer loop as the widest band has sixteens of cells, four to sixteen: the others leave, and the
// barrier does without them.  148 layers, rows of 4097 cells: 105 to 117 us at bands of 1 and of 76 cells on average (the
// layers 55 and 75, the walk 30, records, least total and sizes 15); a loop whose lanes read records and cells from LDS in
// turn took 108 and 137, and 5 more for a second launch that left at once (four waves for narrow bands, sixteen for wide).
// With the shift from row to row in the records, and one clamp between the cells of +inf in the place of a minimum and an
// addition: 140 -> 130 us on the GPT-2-shaped set's table (with the step's look-up), the whole allocation of 148 layers of
// 20 thousand entries 209 -> 195.
constexpr uint32_t BANDED_THREADS = 1024;
constexpr uint32_t BAND_FEW = 8;               // records of a layer that a lane takes one after another where the band is wide
constexpr uint32_t BAND_LIVE_CAP = 2048;       // live records held in LDS at a time
constexpr uint32_t BAND_CELLS = 12288;         // row cells held in LDS (96 KB); two of the longest rows fit
static_assert(2u * DP_ROW_MAX <= BAND_CELLS, "two rows fit");

// Rows and layers as the recurrence sees them: first cell, last cell - first cell, first of the row's cells among all
// rows' cells, first of layer r's live records among all layers'.
struct BandRow { uint32_t lo, span, at, rec; };
__device__ __forceinline__ BandRow band_row(const uint4& v) {
    BandRow b;
    b.lo = __builtin_amdgcn_readfirstlane(v.x); b.span = __builtin_amdgcn_readfirstlane(v.y);
    b.at = __builtin_amdgcn_readfirstlane(v.z); b.rec = __builtin_amdgcn_readfirstlane(v.w);
    return b;
}

// Minimum over the live records of the lane's row, of which there are at most 4 B, for one cell.  Addresses in LDS: `at` the
// cell's own place in its row, counted from the previous row's first cell; a record's z leads from there to its source; what lies
// outside the row becomes one of the cells of +inf before it and behind it, `below` and `beyond`.
__device__ __forceinline__ int med3_i32(int a, int b, int c) {
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
template <int K4, int B>
__device__ __forceinline__ void band_ask(uint32_t z, uint32_t at, int below, int beyond, double (&t)[B][4]) {
    uint32_t q[4];
    row_addr_sub4<4 * K4>(at, z, q);
#pragma unroll
    for (int u = 0; u < 4; ++u) t[K4][u] = *(lds_cdouble_ptr)(uintptr_t)(uint32_t)med3_i32((int)q[u], below, beyond);
}
template <int B>
__device__ __forceinline__ double band_records(uint32_t z, double err, double one, uint32_t at, int below, int beyond) {
    double t[B][4], m[B];
    band_ask<0>(z, at, below, beyond, t);
    if constexpr (B > 1) band_ask<1>(z, at, below, beyond, t);
    if constexpr (B > 2) band_ask<2>(z, at, below, beyond, t);
    if constexpr (B > 3) band_ask<3>(z, at, below, beyond, t);
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
    return min_over_rows(best);
}

__global__ __launch_bounds__(BANDED_THREADS) void k_dp_banded(AllocBuffers ab, DpLists dl, BandBuffers bb, double* rows_g,
                                                              uint32_t rstride, int32_t err_infeasible, int32_t err_nonfinite, StepLookup sl) {
    constexpr uint32_t MAX_WAVES = BANDED_THREADS / 64;
    __shared__ double rows_before[BAND_CELLS + 1u];       // a cell of +inf, then the rows, each with one behind it
    double* const rows = rows_before + 1u;
    __shared__ uint4 recs[BAND_LIVE_CAP];                 // error bits, the way from a cell's own place to its source in bytes
    __shared__ uint4 s_row[BAND_MAX_L + 1];
    __shared__ double s_val[BAND_MAX_L + 1];              // the path's value per row
    __shared__ uint8_t s_k[BAND_MAX_L];                   // the path's live record per layer
    __shared__ uint8_t s_first[BAND_MAX_L + 1];           // first live record of a layer
    __shared__ uint32_t su[16];
    __shared__ unsigned long long su64[16];
    __shared__ double sd[MAX_WAVES];
    __shared__ uint32_t sc[MAX_WAVES];
    __shared__ uint32_t s_bad;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t L = ab.L, J = ab.J, cap = ab.cap;
    if (tid == 0) s_bad = 0u;
    __syncthreads();
    const uint32_t NWAVES = min(max((bb.info[0] + 16u) / 16u, 4u), MAX_WAVES), T = NWAVES * 64u;
    if (wave >= NWAVES) return;
    // rows and records: running sums over the layers
    uint32_t cells = 0u, live_total = 0u;
    for (uint32_t r0 = 0u; r0 <= L; r0 += T) {
        const uint32_t r = r0 + tid;
        const bool in = r <= L;
        const uint32_t lo = in ? min(bb.lo[r], cap) : 0u, hi = in ? max(lo, min(bb.hi[r], cap)) : 0u;
        const uint32_t live = r < L ? bb.live[r] : 0u, cnt = min(live >> 8, 64u);
        if (r < L && dl.bad[r]) s_bad = 1u;
        uint32_t ct, lt;
        const uint32_t at = cells + block_exclusive_scan<uint32_t>(in ? hi - lo + 2u : 0u, su, &ct, NWAVES);
        const uint32_t rec = live_total + block_exclusive_scan<uint32_t>(cnt, su, &lt, NWAVES);
        if (in) { s_row[r] = make_uint4(lo, hi - lo, at, rec); s_first[r] = (uint8_t)(live & 0xFFu); }
        cells += ct; live_total += lt;
    }
    // (a lane without a record takes the way of whatever stands behind its layer's: for the last layer that is loaded, this)
    for (uint32_t x = tid; x < BAND_LIVE_CAP; x += T) recs[x] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    const bool any_bad = s_bad != 0u, hopeless = bb.info[4] != 0u;
    const uint32_t wr = min(cap + 2u, BAND_CELLS / 2u - 1u);   // cells per row buffer when only two rows are kept
    const bool all = cells <= BAND_CELLS;

    // the records of layers [a, b) into LDS, eight layers' loads in flight per wave
    auto load_records = [&](uint32_t a, uint32_t b) {
        const uint32_t first = s_row[a].w;
        for (uint32_t i0 = a + wave * 8u; i0 < b; i0 += NWAVES * 8u) {
            double e[8];
            uint32_t w[8], at[8], shift[8];
            bool in[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t i = min(i0 + (uint32_t)u, b - 1u);
                const uint32_t rec = s_row[i].w, cnt = s_row[i + 1u].w - rec;
                in[u] = i0 + (uint32_t)u < b && lane < cnt;
                at[u] = rec - first + lane;
                shift[u] = s_row[i + 1u].x - s_row[i].x;
                const size_t o = in[u] ? (size_t)i * J + min((uint32_t)s_first[i] + lane, J - 1u) : 0;
                e[u] = dl.e[2 * o]; w[u] = dl.w[o];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (in[u]) recs[at[u]] = make_uint4((uint32_t)__double2loint(e[u]), (uint32_t)__double2hiint(e[u]), 8u * (shift[u] - w[u]), 0u);
        }
    };
    int32_t st = any_bad ? err_nonfinite : hopeless ? err_infeasible : 0;
    uint32_t at_last = 0u;                                // where row L's cells are
    uint32_t loaded = 0u;                                 // first layer of the records in LDS
    if (st == 0) {
        if (tid == 0) {
            rows[-1] = DP_INF; rows[0] = 0.0; rows[1] = DP_INF;
            if (!all) { rows[wr] = DP_INF; rows_g[0] = 0.0; }      // (the second buffer starts behind this one)
        }
        double one = 1.0;
        asm volatile("" : "+v"(one));      // keep 1.0 in a vector register pair
        const uint32_t k = (lane & 15u) * 4u + (lane >> 4);     // this lane's record
        uint32_t i = 0u;
        while (i < L) {
            // a group of layers whose live records fit LDS (at least one layer: a list has at most 64 records)
            const uint32_t g0 = s_row[i].w;
            uint32_t i1 = L;
            if (live_total - g0 > BAND_LIVE_CAP) {
                uint32_t lo = i + 1u, hi = L;              // largest end whose records fit
                while (lo < hi) {
                    const uint32_t mid = (lo + hi + 1u) >> 1;
                    if (s_row[mid].w - g0 <= BAND_LIVE_CAP) lo = mid; else hi = mid - 1u;
                }
                i1 = lo;
            }
            load_records(i, i1);
            loaded = i;
            __syncthreads();
            // the record of this lane among n from `rec` on (beyond the last: one that changes no minimum)
            auto record = [&](uint32_t rec, uint32_t n) {
                uint4 r = recs[min(rec - g0 + k, BAND_LIVE_CAP - 1u)];
                r.y = k < n ? r.y : 0x7FF00000u;
                r.x = k < n ? r.x : 0u;
                return r;
            };
            BandRow p = band_row(s_row[i]), c = band_row(s_row[i + 1u]);
            uint4 R = record(p.rec, c.rec - p.rec);
            BandRow nx = band_row(s_row[min(i + 2u, i1)]);
            for (; i < i1; ++i) {
                const uint32_t n = c.rec - p.rec, z = R.z;
                const double err = rec_err(R);
                // the next layer's record and the row after that, asked for now: off the critical path
                const uint4 after = s_row[min(i + 3u, i1)];
                R = record(c.rec, nx.rec - c.rec);
                const uint32_t prow = all ? p.at : (i & 1u) * (wr + 1u), crow = all ? c.at : ((i + 1u) & 1u) * (wr + 1u);
                double* out = all ? nullptr : rows_g + (size_t)(i + 1u) * rstride;
                const uint32_t row = lds_addr(rows + prow);
                const int below = (int)row - 8, beyond = (int)(row + 8u * (p.span + 1u));
                if (n <= BAND_FEW && c.span + 1u >= NWAVES * 16u) {
                    // few records and more cells than the waves have sixteens: a cell a lane, the records one after another
                    for (uint32_t c0 = wave * 64u; c0 <= c.span + 1u; c0 += NWAVES * 64u) {
                        const uint32_t cell = c0 + lane, at = row + 8u * cell;
                        double best = DP_INF;
                        for (uint32_t j = 0; j < n; ++j) {
                            const int from = (int)((j & 3u) * 16u + (j >> 2));             // (the lane that holds record j)
                            const double e = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(err), from),
                                                              __builtin_amdgcn_readlane(__double2loint(err), from));
                            const int q = med3_i32((int)(at + (uint32_t)__builtin_amdgcn_readlane((int)z, from)), below, beyond);
                            best = min_f64(best, *(lds_cdouble_ptr)(uintptr_t)(uint32_t)q + e);
                        }
                        if (cell <= c.span + 1u) {
                            rows[crow + cell] = cell <= c.span ? best : DP_INF;
                            if (out && cell <= c.span) out[cell] = best;
                        }
                    }
                } else {
                    for (uint32_t c0 = wave * 16u; c0 <= c.span + 1u; c0 += NWAVES * 16u) {
                        const uint32_t cell = c0 + (lane & 15u), at = row + 8u * cell;
                        double best;
                        if (n <= 16u) best = band_records<1>(z, err, one, at, below, beyond);
                        else if (n <= 32u) best = band_records<2>(z, err, one, at, below, beyond);
                        else if (n <= 48u) best = band_records<3>(z, err, one, at, below, beyond);
                        else best = band_records<4>(z, err, one, at, below, beyond);
                        if (lane < 16u && cell <= c.span + 1u) {
                            rows[crow + cell] = cell <= c.span ? best : DP_INF;
                            if (out && cell <= c.span) out[cell] = best;
                        }
                    }
                }
                lds_barrier();                             // the next layer reads this row (and the next group overwrites the records)
                p = c; c = nx; nx = band_row(after);
            }
        }
        at_last = all ? s_row[L].z : (L & 1u) * (wr + 1u);
    }
    // ---- least total of the last row, smallest cost attaining it
    double best = DP_INF;
    uint32_t bc = 0xFFFFFFFFu;
    if (st == 0) {
        const uint32_t llo = s_row[L].x, span = s_row[L].y;
        for (uint32_t x = tid; x <= span; x += T) {
            const double v = rows[at_last + x];
            if (v < best) { best = v; bc = llo + x; }      // ascending: keeps the smallest cost
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            const double ov = __shfl_xor(best, d, 64);
            const uint32_t oc = __shfl_xor(bc, d, 64);
            if (ov < best || (ov == best && oc < bc)) { best = ov; bc = oc; }
        }
        if (lane == 0) { sd[wave] = best; sc[wave] = bc; }
        __syncthreads();
        for (uint32_t v = 0; v < NWAVES; ++v)
            if (sd[v] < best || (sd[v] == best && sc[v] < bc)) { best = sd[v]; bc = sc[v]; }
        if (!(best < DP_INF)) st = err_infeasible;
    }
    if (tid == 0) *ab.status = st;
    if (st != 0) {                                         // (the same in every thread)
        for (uint32_t i = tid; i < L; i += T) { ab.j_out[i] = 0; ab.K_out[i] = 0; }
        for (uint32_t i = tid; i <= L; i += T) ab.offsets_out[i] = 0;
        step_lookup(sl, T);
        return;
    }
    // ---- the walk back, in groups of layers whose records, and staged rows, fit LDS
    if (tid == 0) s_val[L] = best;
    uint32_t rel = bc - s_row[L].x;                        // the path's cell, counted from its row's first
    double val = best;
    uint32_t hi = L;
    while (hi > 0u) {
        uint32_t lo = 0u;
        if (s_row[hi].w > BAND_LIVE_CAP || (!all && s_row[hi].z > BAND_CELLS)) {
            uint32_t a = 0u, b = hi - 1u;                  // smallest start whose records and rows fit
            while (a < b) {
                const uint32_t mid = (a + b) >> 1;
                if (s_row[hi].w - s_row[mid].w <= BAND_LIVE_CAP && (all || s_row[hi].z - s_row[mid].z <= BAND_CELLS)) b = mid; else a = mid + 1u;
            }
            lo = a;
        }
        __syncthreads();                                   // (also: the rows written to memory are there)
        const uint32_t row0 = all ? 0u : s_row[lo].z;      // the cells in LDS start here
        if (lo < loaded || !all) {
            load_records(lo, hi);
            loaded = lo;
        }
        const uint32_t rec0 = s_row[loaded].w;
        if (!all) {
            for (uint32_t r = lo + wave; r < hi; r += NWAVES) {
                const uint4 d = s_row[r];
                const double* src = rows_g + (size_t)r * rstride;
                for (uint32_t x = lane; x <= d.y; x += 64u) rows[d.z - row0 + x] = src[x];
            }
        }
        __syncthreads();
        if (wave == 0u) {
            BandRow c = band_row(s_row[hi]), p = band_row(s_row[hi - 1u]), next = band_row(s_row[hi - 1u > lo ? hi - 2u : lo]);
            uint4 r = recs[p.rec - rec0 + min(lane, max(c.rec - p.rec, 1u) - 1u)];
            for (uint32_t i = hi; i-- > lo;) {
                const uint32_t n = c.rec - p.rec;
                const uint4 after = s_row[i > lo + 1u ? i - 2u : lo];
                // the record of the layer before (`next` is its row), asked for now, as the row before that
                const uint4 rn = recs[next.rec - rec0 + min(lane, max(p.rec - next.rec, 1u) - 1u)];
                const uint32_t src = rel + (uint32_t)((int)r.z >> 3);            // (counted from the row's first cell)
                const bool in = lane < n && src <= p.span;
                const double v = rows[p.at - row0 + (in ? src : 0u)];
                const uint64_t hit = ballot(in && v + rec_err(r) == val);
                const uint32_t k = hit ? (uint32_t)__builtin_ctzll(hit) : 0u;  // (there is one)
                if (lane == k) { s_k[i] = (uint8_t)k; s_val[i] = v; }
                rel = (uint32_t)__builtin_amdgcn_readlane((int)src, (int)k);
                val = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), (int)k),
                                       __builtin_amdgcn_readlane(__double2loint(v), (int)k));
                r = rn; c = p; p = next; next = band_row(after);
            }
        }
        hi = lo;
    }
    __syncthreads();
    // ---- winners, sizes and offsets, in parallel
    unsigned long long carry = 0ull;
    for (uint32_t i0 = 0u; i0 < L; i0 += T) {
        const uint32_t i = i0 + tid;
        unsigned long long K = 0ull;
        uint32_t j = 0u;
        if (i < L) {
            const size_t o = (size_t)i * J + min((uint32_t)s_first[i] + (uint32_t)s_k[i], J - 1u);
            const uint32_t jj = dl.jj[o];
            const double from = s_val[i], to = s_val[i + 1u];
            j = jj >> 8;
            // the lowest member of the run whose rounded total is the same (NaN for a single: never equal)
            if (from + dl.e[2 * o + 1] == to) {
                const uint32_t jlo = jj & 0xFFu;
                --j;
                while (j > jlo && from + ab.E[(size_t)i * J + j - 1u] == to) --j;
            }
            j = min(j, J - 1u);
            K = ab.Kout[(size_t)i * J + j];
        }
        unsigned long long total;
        const unsigned long long off = carry + block_exclusive_scan<unsigned long long>(K, su64, &total, NWAVES);
        if (i < L) { ab.j_out[i] = (int32_t)j; ab.K_out[i] = K; ab.offsets_out[i] = off; }
        carry += total;
    }
    if (tid == 0) ab.offsets_out[L] = carry;
    step_lookup(sl, T);
}

}  // namespace kimad
