// Knapsack allocation by a tree of segments (paper Appendix C; Section 3.2, Eq. optimisation).
//
// The recurrence of k_alloc.h is a chain of L steps, because its totals are sums from the left.  The allocation itself is not:
// least totals of segments of layers, summed and joined in any order, name the same sizes unless two allocations lie within
// rounding of each other.  So:
//
//   k_dp_segments  least totals of every segment of layers for every cost, all segments side by side, and the candidate lists;
//   k_dp_join      least totals of two neighbours together: out[c] = min over a of A[a] + B[c - a]; a launch per level;
//   k_dp_path      from the whole down to the layers: what each half spends, and at every choice whether the second best lies
//                  beyond the rounding of any order of summation.  If it does throughout, the sizes are written out; if not, the
//                  chain (k_dp_chain, k_dp_walk), which otherwise leaves after one load, decides.
//
// Why the result is the chain's, bit for bit.  Let p be the allocation found, and every other one (as a choice of list entries)
// larger in exact arithmetic by more than twice what a sum of L terms may be off.  The chain's total of an allocation is its
// sum from the left, so p alone attains its least total; a row's cell on p's way has no other way that attains its value, or
// that way with the rest of p would attain p's total too (fp64 addition is monotone).  So the chain walks back along p.  An
// entry dearer than another of its layer and no better is left out: the same way with the other one ends at a smaller cost with no
// greater total, and the chain takes the smallest cost that attains the least total.  Which member of a run of equal costs the
// chain names hangs on the rounded sums from the left, which are formed for p where they may matter.
//
// Costs are counted from the layers' cheapest entries on: what those leave of the capacity is the room, and nothing costs more.
#pragma once
#include "common.h"
#include "k_alloc.h"
#include "k_alloc_band.h"
#include "last_of_cost.h"

namespace kimad {

constexpr uint32_t TREE_MAX_L = 1024, TREE_MAX_SEGMENTS = 64, TREE_LAYERS = 16;     // layers, segments, layers of a segment
static_assert(TREE_MAX_SEGMENTS * TREE_LAYERS == TREE_MAX_L, "every layer has a place");
constexpr uint32_t TREE_NO_ROOM = 0xFFFFFFFFu;
enum : uint32_t { TREE_UNSURE = 1u, TREE_BAD = 2u, TREE_NEAR = 4u, TREE_AT_ONCE = 8u };         // head[2]

// An entry of the list of a layer that has a choice, as k_dp_path takes it.
struct TreeEntry {
    double e, before;      // error; of the run's next member that has another one (NaN: there is none)
    uint32_t w;            // cost beyond the layer's cheapest; 0xFFFFFFFF: no entry
    uint32_t place;        // place in the layer's list (DpLists) | the run's lowest member of this error << 16
    uint32_t K;
    uint32_t pad;
};
// A layer all of whose sizes cost the same: its best entry, and how much worse the next best and the run's next member are.
struct TreeSingle {
    double next, before;   // (+inf, NaN: there is none)
    uint32_t place, K;     // place as above; 0xFFFFFFFF: the layer has a choice
};

struct TreeBuffers {
    double* vec;           // [2 S][pitch] least totals of node k's layers by cost; node 1 is the whole, 2 k and 2 k + 1 the halves of k
    uint32_t* hi;          // [2 S] the largest cost of a node
    TreeEntry* entry;      // [S][TREE_LAYERS][64] a segment's layers, in the order of its rows
    uint32_t* layer;       // [S][TREE_LAYERS] which they are,
    uint32_t* row_hi;      // [S][TREE_LAYERS] and the largest cost of the row behind each
    TreeSingle* single;    // [L]
    uint32_t* at;          // [L] the path's entry: its place in the layer's list
    uint32_t* head;        // [0] room, [1] segments done, [2] TREE_UNSURE .., [3] the chain decides, [4] layers with a choice
    double* rows;          // [L][pitch] a segment's least totals behind each of its layers (k_dp_chain's rows)
    uint32_t pitch;
    uint32_t S;            // segments, a power of two
};

// The layers that have a choice, for a workgroup of TREE_MAX_L threads: their number, the room, and this thread's layer's number among them.
struct TreeLayers {
    uint32_t number, reach, count, room;               // number 0xFFFFFFFF: no choice
    __device__ __forceinline__ void find(const AllocBuffers& ab, uint32_t (*scratch)[16]) {
        const uint32_t i = threadIdx.x, wave = i >> 6;
        uint32_t k0 = 0u, k1 = 0u;
        if (i < ab.L) { k0 = ab.Ktab[(size_t)i * ab.J]; k1 = ab.Ktab[(size_t)i * ab.J + ab.J - 1u]; }
        const uint32_t w0 = units_of(k0, ab.unit), w1 = units_of(k1, ab.unit);
        const uint64_t choice = ballot(w1 != w0);
        const uint32_t least = wave_scan_add_u32(min(w0, ab.cap + 1u));            // (1024 layers of at most 4225)
        if (lane_id() == 63u) { scratch[0][wave] = (uint32_t)__popcll(choice); scratch[1][wave] = least; }
        __syncthreads();
        uint32_t before = 0u, sum = 0u;
        count = 0u;
#pragma unroll
        for (uint32_t v = 0; v < TREE_MAX_L / 64u; ++v) {
            if (v < wave) before += scratch[0][v];
            count += scratch[0][v];
            sum += scratch[1][v];
        }
        number = w1 != w0 ? before + mbcnt(choice) : 0xFFFFFFFFu;
        reach = w1 - w0;
        room = sum > ab.cap ? TREE_NO_ROOM : ab.cap - sum;
    }
};

// Of a layer's list (dp_list, by one wave), what is neither dearer nor worse than another entry, and its place among that.
struct TreeKept { bool keep; uint32_t at, w; uint64_t kept; };
__device__ __forceinline__ TreeKept tree_kept(const DpList& d) {
    const uint32_t lane = lane_id();
    double least = d.start ? d.e_last : DP_INF;
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
        const double o = __shfl_up(least, s, 64);
        if ((int)lane >= s) least = fmin(least, o);
    }
    const double before = __shfl_up(least, 1, 64);
    TreeKept t;
    t.keep = d.start && (lane == 0u || d.e_last < before);
    t.kept = ballot(t.keep);
    t.at = mbcnt(t.kept);
    t.w = d.w - (uint32_t)__builtin_amdgcn_readfirstlane((int)d.w);
    return t;
}
// Of a run of equal costs, its lowest member of the last one's very error: whatever the sums from the left, theirs are the same, so
// the chain names no higher one.  And the error of the next member down, which may come to the same total by rounding (NaN: none).
// (Grids name many a size of a short layer twice, and that alone is no reason to form the totals from the left.)
struct TreeRun { uint32_t low; double before; };
__device__ __forceinline__ TreeRun tree_run(const DpList& d) {
    const uint32_t last = d.last & 63u;
    TreeRun r;
    r.low = last - min(last, (uint32_t)__clzll((long long)~(d.same << (63u - last))));       // (the run's first is not marked)
    const double below = __shfl(d.e, (int)((r.low - 1u) & 63u), 64);
    r.before = r.low > lane_id() ? below : __longlong_as_double(0x7FF8000000000000ll);
    return r;
}

// Least totals of the segments, by workgroup s < S; the lists, a wave a layer, by the others.
// Bound by the LDS reads and instructions of a row's cells and a layer's entries (TREE_FEW), and by the way there: the sizes, the
// lists.
constexpr uint32_t SEGMENT_THREADS = 1024;
template <uint32_t MAXC>
__global__ __launch_bounds__(SEGMENT_THREADS) void k_dp_segments(AllocBuffers ab, DpLists dl, TreeBuffers tb) {
    constexpr uint32_t NT = SEGMENT_THREADS, WAVES = NT / 64u, CPT = (MAXC + NT - 1u) / NT;
    constexpr uint32_t U = CPT <= 1u ? 8u : 4u;          // entries whose cells are asked for together
    static_assert(WAVES == TREE_LAYERS && NT == TREE_MAX_L, "a wave a layer, a thread a layer");
    __shared__ double rows[2][2u * MAXC];                // MAXC cells of +inf before cost 0: what a cell cannot afford
    __shared__ uint4 recs[WAVES][64];                    // entries: error bits, cost as a distance in bytes
    __shared__ uint32_t rec_n[WAVES], rec_hi[WAVES];
    __shared__ uint32_t layer[TREE_LAYERS], reach[TREE_LAYERS], sorted[TREE_LAYERS];
    __shared__ uint32_t su[2][16];
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    if (blockIdx.x >= tb.S) {
        const uint32_t i = (blockIdx.x - tb.S) * WAVES + wave;
        if (i >= ab.L) return;
        const DpList d = dp_list(ab, i, lane);
        dp_list_store(ab, dl, i, lane, d);
        double largest = d.start ? fabs(d.e_last) : 0.0;
#pragma unroll
        for (int s = 32; s > 0; s >>= 1) largest = fmax(largest, __shfl_xor(largest, s, 64));
        if (lane == 0u) dl.habs[i] = largest;
        const bool choice = units_of(ab.Ktab[(size_t)i * ab.J], ab.unit) != units_of(ab.Ktab[(size_t)i * ab.J + ab.J - 1u], ab.unit);
        const TreeKept t = tree_kept(d);
        const TreeRun run = tree_run(d);
        const uint64_t kept = t.kept;
        const int last = kept ? 63 - __builtin_clzll(kept) : 0;                    // the best entry's lane, and the next best's
        const uint64_t others = kept & ~(1ull << last);
        const double next = __shfl(d.e_last, others ? 63 - __builtin_clzll(others) : 0, 64);
        if (lane == (uint32_t)last) {
            TreeSingle one;
            one.next = others ? next - d.e_last : DP_INF;
            one.before = run.before - d.e_last;
            one.place = choice || !kept ? 0xFFFFFFFFu : mbcnt(d.starts) | (run.low << 16);
            one.K = ab.Kout[(size_t)i * ab.J + min(run.low, ab.J - 1u)];
            tb.single[i] = one;
        }
        return;
    }
    const uint32_t s = blockIdx.x, ahead = ab.info[INFO_AHEAD];
    for (uint32_t x = tid; x < 4u * MAXC; x += NT) (&rows[0][0])[x] = DP_INF;
    TreeLayers all;
    all.find(ab, su);
    const uint32_t room = all.room;
    if (ahead) {
        // whole rows at once: they are made ready for the chain, and nothing else looks at a tree that has no room
        for (uint32_t r = s * WAVES + wave; r <= ab.L; r += tb.S * WAVES) dp_fill_row(ab, tb.rows, tb.pitch, 0u, r, lane, 64u);
        if (s) return;
        if (tid < 5u) tb.head[tid] = tid == 0u ? TREE_NO_ROOM : tid == 2u ? (uint32_t)TREE_AT_ONCE : tid == 3u ? 1u : 0u;
        if (tid < 4u) ab.flags[tid] = tid == 1u ? ab.first_ticket : 0u;
        if (tid < INFO_REPORT) ab.info[tid] = tid == INFO_ROUTE ? ROUTE_TREE : tid == INFO_HOW ? HOW_ROWS | HOW_AT_ONCE : 0u;
        return;
    }
    if (s == 0u && tid < 5u) tb.head[tid] = tid == 0u ? room : tid == 4u ? all.count : 0u;
    if (s == 0u) alloc_report(ab, ROUTE_TREE, tid);
    if (room == TREE_NO_ROOM) return;
    // (the host has chosen S so that a segment has at most TREE_LAYERS)
    const uint32_t per = min((all.count + tb.S - 1u) / tb.S, TREE_LAYERS), first = min(s * per, all.count), m = min(per, all.count - first);
    {
        const uint32_t x = all.number - first;
        if (all.number >= first && all.number != 0xFFFFFFFFu && x < m) { layer[x] = tid; reach[x] = all.reach; }
    }
    __syncthreads();
    // the layers that reach least first: the row is short as long as only they are in it
    if (tid < m) {
        uint32_t rank = 0u;
        for (uint32_t y = 0; y < m; ++y) rank += reach[y] < reach[tid] || (reach[y] == reach[tid] && y < tid) ? 1u : 0u;
        sorted[rank] = layer[tid];
        tb.layer[s * TREE_LAYERS + rank] = layer[tid];
    }
    __syncthreads();
    if (wave < m) {
        const uint32_t i = (uint32_t)__builtin_amdgcn_readfirstlane((int)sorted[wave]);
        const DpList d = dp_list(ab, i, lane);
        const TreeKept t = tree_kept(d);
        const TreeRun run = tree_run(d);
        const bool fits = t.keep && t.w <= room;                                   // (costs ascend: the first ones)
        const uint32_t n = (uint32_t)__popcll(ballot(fits));
        TreeEntry* out = tb.entry + ((size_t)s * TREE_LAYERS + wave) * 64u;
        if (fits) {
            recs[wave][t.at] = make_uint4((uint32_t)__double2loint(d.e_last), (uint32_t)__double2hiint(d.e_last), 8u * t.w, 0u);
            TreeEntry x;
            x.e = d.e_last;
            x.before = run.before;
            x.w = t.w; x.place = mbcnt(d.starts) | (run.low << 16); x.K = ab.Kout[(size_t)i * ab.J + min(run.low, ab.J - 1u)]; x.pad = 0u;
            out[t.at] = x;
            if (t.at == n - 1u) rec_hi[wave] = t.w;
        }
        if (lane >= n) {
            recs[wave][lane] = make_uint4(0u, 0x7FF00000u, 8u * MAXC, 0u);
            out[lane].w = 0xFFFFFFFFu;
        }
        if (lane == 0u) { rec_n[wave] = n; if (n == 0u) rec_hi[wave] = 0u; }
    }
    __syncthreads();
    uint32_t hi = 0u, cur = 0u;                           // the row's largest cost, and which of the two it is
    if (m == 0u && tid == 0u) rows[0][MAXC] = 0.0;
    for (uint32_t u = 0; u < m; ++u) {
        const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)rec_n[u]), i = (uint32_t)__builtin_amdgcn_readfirstlane((int)sorted[u]);
        const uint4 mine = recs[u][lane];
        hi = min(room, hi + (uint32_t)__builtin_amdgcn_readfirstlane((int)rec_hi[u]));
        double* out = tb.rows + (size_t)i * tb.pitch;
        if (tid == 0u) tb.row_hi[s * TREE_LAYERS + u] = hi;
        if (u == 0u) {
            // the first layer's row: its entries, of equal costs the last (two lanes' stores to one cell have no order)
            if (tid < n && last_of_cost(tid, n, [&](uint32_t k) { return recs[0][k].z; })) rows[0][MAXC + mine.z / 8u] = rec_err(mine);
            __syncthreads();
            for (uint32_t c = tid; c <= hi; c += NT) out[c] = rows[0][MAXC + c];
            continue;
        }
        const double* prev = rows[cur] + MAXC;
        double* next = rows[cur ^ 1u] + MAXC;
        const uint32_t w8 = mine.z;
        const uint32_t base = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid & ~63u));
        auto step = [&](auto nq) {
            constexpr uint32_t NQ = decltype(nq)::value;
            // (threads beyond the longest row read its last cell)
            const uint32_t from = lds_addr(prev) + 8u * tid, far = lds_addr(prev) + 8u * min(tid + (NQ - 1u) * NT, MAXC - 1u);
            double best[NQ];
#pragma unroll
            for (uint32_t q = 0; q < NQ; ++q) best[q] = DP_INF;
            for (uint32_t k0 = 0; k0 < n; k0 += U) {
                double t[U][NQ];
#pragma unroll
                for (uint32_t k = 0; k < U; ++k) {
                    const uint32_t cost = (uint32_t)__builtin_amdgcn_readlane((int)w8, (int)(k0 + k));
#pragma unroll
                    for (uint32_t q = 0; q < NQ; ++q)
                        t[k][q] = *(lds_cdouble_ptr)(uintptr_t)(NQ * NT > MAXC && q == NQ - 1u ? far - cost : from - cost + 8u * q * NT);
                }
#pragma unroll
                for (uint32_t k = 0; k < U; ++k) {
                    const double e = __hiloint2double(__builtin_amdgcn_readlane((int)mine.y, (int)(k0 + k)), __builtin_amdgcn_readlane((int)mine.x, (int)(k0 + k)));
#pragma unroll
                    for (uint32_t q = 0; q < NQ; ++q) best[q] = min_f64(best[q], t[k][q] + e);
                }
            }
#pragma unroll
            for (uint32_t q = 0; q < NQ; ++q) {
                const uint32_t c = tid + q * NT;
                if (c <= hi) { next[c] = best[q]; out[c] = best[q]; }
            }
        };
        // (cells beyond the row's largest cost stay +inf)
        if (CPT > 4u && base + 4u * NT <= hi) step(std::integral_constant<uint32_t, CPT>{});
        else if (CPT > 2u && base + 2u * NT <= hi) step(std::integral_constant<uint32_t, CPT < 4u ? CPT : 4u>{});
        else if (CPT > 1u && base + NT <= hi) step(std::integral_constant<uint32_t, CPT < 2u ? CPT : 2u>{});
        else if (base <= hi) step(std::integral_constant<uint32_t, 1u>{});
        cur ^= 1u;
        lds_barrier();
    }
    __syncthreads();
    const double* row = rows[cur] + MAXC;
    double* out = tb.vec + (size_t)(tb.S + s) * tb.pitch;
    for (uint32_t c = tid; c <= hi; c += NT) out[c] = row[c];
    if (tid == 0u) tb.hi[tb.S + s] = hi;
}

// Two neighbours together: node k of the level's nodes k = first + blockIdx.y, T costs.  A lane looks after R neighbouring costs; T / R
// lanes share a part of the costs that the first half may take, four at a time: eight values are read for 4 R sums, and R + 3 of B's
// stay for the next four.
// Bound by the additions and minima, and on rows of 4097 cells with T = 16 by what every workgroup brings to LDS.
// (us, nodes of 4097 cells, under the profiler: eight, T = 64 and R = 4, 21.9 with the rows brought one load at a time and 17.7 with
// eight, R = 8 16.7; four, T = 16 19.6 and 14.2, T = 64 and R = 8 11.8; two, T = 16 14.0 and 9.6, T = 32 9.3.)
constexpr uint32_t JOIN_THREADS = 256;
template <uint32_t MAXC, uint32_t T, uint32_t R>
__global__ __launch_bounds__(JOIN_THREADS) void k_dp_join(TreeBuffers tb, uint32_t first) {
    constexpr uint32_t LANES = T / R, PARTS = JOIN_THREADS / LANES, OFF = T + 11u;
    static_assert(T % 16u == 0 && R % 4u == 0 && OFF % 4u == 3u, "a lane's costs, and what it reads of B, start at whole quads");
    __shared__ __align__(16) double A[MAXC + 8u];
    __shared__ __align__(16) double B[OFF + MAXC + T + 5u];
    __shared__ double red[JOIN_THREADS / 64u][T];
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const uint32_t k = first + blockIdx.y, c0 = (gridDim.x - 1u - blockIdx.x) * T;      // (those with most to do come first)
    const uint32_t room = tb.head[0];
    if (room == TREE_NO_ROOM) return;
    const uint32_t ha = tb.hi[2u * k], hb = tb.hi[2u * k + 1u], hk = min(room, ha + hb);
    if (c0 > hk) return;
    if (c0 == 0u && tid == 0u) tb.hi[k] = hk;
    const uint32_t top = min(c0 + T - 1u, MAXC - 1u);                        // (hk < MAXC)
    const uint32_t a_lo = (c0 > hb ? c0 - hb : 0u) & ~3u, a_hi = min(ha, min(top, hk));
    const double* va = tb.vec + (size_t)(2u * k) * tb.pitch;
    const double* vb = tb.vec + (size_t)(2u * k + 1u) * tb.pitch;
    // (eight loads of each at a time)
    for (uint32_t x0 = tid; x0 < max(a_hi + 4u, OFF + top + 2u) - a_lo; x0 += 8u * JOIN_THREADS) {
        double ra[8], rb[8];
#pragma unroll
        for (uint32_t u = 0; u < 8u; ++u) {
            const uint32_t x = x0 + u * JOIN_THREADS, a = a_lo + x, b = x - OFF;
            ra[u] = va[min(a, ha)];
            rb[u] = vb[x >= OFF ? min(b, hb) : 0u];
        }
#pragma unroll
        for (uint32_t u = 0; u < 8u; ++u) {
            const uint32_t x = x0 + u * JOIN_THREADS, a = a_lo + x, b = x - OFF;
            if (a < a_hi + 4u) A[a] = a <= ha ? ra[u] : DP_INF;
            if (x < OFF + top + 2u - a_lo) B[x] = x >= OFF && b <= hb ? rb[u] : DP_INF;
        }
    }
    __syncthreads();
    const uint32_t l = tid % LANES, part = tid / LANES, c = c0 + R * l;
    const uint32_t quads = (a_hi - a_lo) / 4u + 1u, per = (quads + PARTS - 1u) / PARTS;
    const uint32_t a0 = a_lo + 4u * part * per, a1 = min(a0 + 4u * per, a_lo + 4u * quads);
    double best[R];
#pragma unroll
    for (uint32_t v = 0; v < R; ++v) best[v] = DP_INF;
    if (a0 < a1) {
        // w[v - u + 3] = B[c + v - a - u]
        const double* bp = B + OFF + c - a0 - 3u;
        double w[R + 4u];
#pragma unroll
        for (uint32_t v = 0; v < R + 4u; v += 2u) {
            const double2 p = *reinterpret_cast<const double2*>(bp + v);
            w[v] = p.x; w[v + 1u] = p.y;
        }
        for (uint32_t a = a0; a < a1; a += 4u) {
            const double2 x0 = *reinterpret_cast<const double2*>(A + a), x1 = *reinterpret_cast<const double2*>(A + a + 2u);
            const double x[4] = {x0.x, x0.y, x1.x, x1.y};
            bp -= 4;
            const double2 n0 = *reinterpret_cast<const double2*>(bp), n1 = *reinterpret_cast<const double2*>(bp + 2);
#pragma unroll
            for (uint32_t u = 0; u < 4u; ++u)
#pragma unroll
                for (uint32_t v = 0; v < R; ++v) best[v] = min_f64(best[v], x[u] + w[v + 3u - u]);
#pragma unroll
            for (uint32_t v = R + 2u; v >= 4u; --v) w[v] = w[v - 4u];
            w[0] = n0.x; w[1] = n0.y; w[2] = n1.x; w[3] = n1.y;
        }
    }
#pragma unroll
    for (uint32_t d = LANES; d < 64u; d <<= 1)
#pragma unroll
        for (uint32_t v = 0; v < R; ++v) best[v] = min_f64(best[v], __shfl_xor(best[v], (int)d, 64));
    if (lane < LANES)
#pragma unroll
        for (uint32_t v = 0; v < R; ++v) red[wave][R * lane + v] = best[v];
    __syncthreads();
    if (tid < T && c0 + tid <= hk) {
        double r = red[0][tid];
#pragma unroll
        for (uint32_t v = 1; v < JOIN_THREADS / 64u; ++v) r = min_f64(r, red[v][tid]);
        tb.vec[(size_t)k * tb.pitch + c0 + tid] = r;
    }
}

// Least of a workgroup's values, where it is, and the second least.
struct Two { double best, second; uint32_t at; };
__device__ __forceinline__ void two_add(Two& t, double v, uint32_t at) {
    t.second = min_f64(t.second, max_f64(t.best, v));
    if (v < t.best) { t.best = v; t.at = at; }
}
__device__ __forceinline__ Two two_wave(const Two& t) {
    Two r;
    r.best = wave_min_f64(t.best);
    const uint64_t who = ballot(t.best == r.best);
    const uint32_t first = who ? (uint32_t)__builtin_ctzll(who) : 0u;
    r.second = wave_min_f64(lane_id() == first ? t.second : t.best);
    r.at = (uint32_t)__builtin_amdgcn_readlane((int)t.at, (int)first);
    return r;
}

// The same for a running minimum over the lanes below and the lane itself.
__device__ __forceinline__ double wave_scan_min_f64(double v) {
    auto from = [](double x, auto ctrl, auto rows) {
        const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), decltype(ctrl)::value, decltype(rows)::value, 0xF, false);
        const int hi = __builtin_amdgcn_update_dpp(0x7FF00000, __double2hiint(x), decltype(ctrl)::value, decltype(rows)::value, 0xF, false);
        return __hiloint2double(hi, lo);                   // (+inf where there is no lane to take it from)
    };
    using std::integral_constant;
    v = min_f64(v, from(v, integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{}));      // row_shr:1, 2, 4, 8
    v = min_f64(v, from(v, integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{}));
    v = min_f64(v, from(v, integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{}));
    v = min_f64(v, from(v, integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{}));
    v = min_f64(v, from(v, integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{}));      // row_bcast:15, 31
    v = min_f64(v, from(v, integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{}));
    return v;
}

// The way down, a workgroup per segment: what the whole's halves spend, the half's halves on the segment's side, ..., and the
// segment's layers from the last one back.  At every choice the second best is looked at.  The nodes that a segment's way passes
// are known beforehand, so their totals (rows of up to 1024 cells, NODES), and its layers' entries, are asked for at once.  The
// segment that is through last makes the offsets.
// A chain of dependent steps: the loads, a minimum of some hundred sums per level, the rows, an LDS read per layer, the
// counter, the offsets, the look-up.
constexpr uint32_t PATH_THREADS = 512;
constexpr uint32_t PATH_STAGE = 12288;             // cells of rows in LDS (a row of the longest kind fits)
constexpr uint32_t PATH_LEVELS = 6;
static_assert(1u << PATH_LEVELS == TREE_MAX_SEGMENTS && PATH_STAGE >= 2u * PATH_LEVELS * 1024u && PATH_STAGE >= DP_ROW_MAX, "the nodes' totals fit");
// Behind ties in a row (alloc_decided) the chain comes at once, and the tree's kernels leave.
// (us of all launches of the allocation, the chain or the band alone, tree and chain, and the chain at once, of 16 and of 64 ratios: 148 layers,
// 1000 cells 72, 118, 84 and 107, 154, 119; 1537 cells 144 in place of 177 by the band, 102, and 183 in place of 170, 139; 4097 cells 183, 302, 230
// and 223, 352, 284; 62 layers, 1000 cells 48, 82, 58.)

// What a segment has found for a layer goes beyond the caches: the segment that is through last reads it.
__device__ __forceinline__ void tree_store(const AllocBuffers& ab, const TreeBuffers& tb, uint32_t i, uint32_t place, uint32_t K) {
    __hip_atomic_store(&tb.at[i], place & 0xFFFFu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&ab.j_out[i], (int32_t)(place >> 16), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&ab.K_out[i], (uint64_t)K, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool NODES>
__global__ __launch_bounds__(PATH_THREADS) void k_dp_path(AllocBuffers ab, DpLists dl, TreeBuffers tb, int32_t err_infeasible, int32_t err_nonfinite,
                                                          StepLookup sl) {
    constexpr uint32_t NT = PATH_THREADS, WAVES = NT / 64u, LR = TREE_LAYERS / WAVES, LT = TREE_MAX_L / NT;
    constexpr uint32_t ROW = NODES ? 1024u : DP_ROW_MAX, PER = (ROW + NT - 1u) / NT;
    __shared__ __align__(16) double stage[PATH_STAGE];         // the nodes' totals, then rows
    __shared__ double least[PER * NT];                         // the least total of the whole's second half up to a cost
    __shared__ double rec_e[TREE_LAYERS][64];
    __shared__ uint32_t rec_w[TREE_LAYERS][64], rec_place[TREE_LAYERS][64], rec_K[TREE_LAYERS][64];
    __shared__ uint64_t rec_near[TREE_LAYERS];                 // entries whose run has a member near the last
    __shared__ uint32_t s_hi[2u * TREE_MAX_SEGMENTS];
    __shared__ Two s_two[2][WAVES];
    __shared__ double sd[16];
    __shared__ uint32_t su[2][16];
    __shared__ uint32_t s_x, s_last, s_state;
    const uint32_t tid = threadIdx.x, lane = lane_id(), wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t L = ab.L, s = blockIdx.x;
    const uint32_t levels = 31u - (uint32_t)__clz((int)tb.S);
    auto node_at = [&](uint32_t lev) { return (tb.S + s) >> (levels - lev); };          // the segment's ancestor, from the whole (lev 0) down
    // ---- what the launches before left, all of it asked for at once (what a node's row holds beyond its largest cost is dropped)
    const uint32_t room = tb.head[0], count = tb.head[4];
    const uint32_t my_hi = tb.hi[min(tid, 2u * tb.S - 1u)];
    double largest = 0.0;
#pragma unroll
    for (uint32_t q = 0; q < LT; ++q) largest += q * NT + tid < L ? dl.habs[q * NT + tid] : 0.0;
    TreeEntry entry[LR];
#pragma unroll
    for (uint32_t q = 0; q < LR; ++q) entry[q] = tb.entry[((size_t)s * TREE_LAYERS + wave + q * WAVES) * 64u + lane];
    const uint32_t my_layer = tb.layer[s * TREE_LAYERS + (lane & (TREE_LAYERS - 1u))], my_row_hi = tb.row_hi[s * TREE_LAYERS + (lane & (TREE_LAYERS - 1u))];
    const uint32_t share = (L + tb.S - 1u) / tb.S;                                       // a share of the layers of one cost
    TreeSingle single[LT];
    uint32_t bad[LT];
#pragma unroll
    for (uint32_t q = 0; q < LT; ++q) {
        const uint32_t i = min(s * share + min(q * NT + tid, share - 1u), L - 1u);
        single[q] = tb.single[i]; bad[q] = dl.bad[i];
    }
    double v[PATH_LEVELS][4];
    if (NODES) {
#pragma unroll
        for (uint32_t lev = 0; lev < PATH_LEVELS; ++lev) {
            if (lev >= levels) continue;
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) v[lev][q] = tb.vec[(size_t)(2u * node_at(lev) + (q >> 1)) * tb.pitch + tid + (q & 1u) * NT];
        }
    }
    if (room == TREE_NO_ROOM && (tb.head[2] & TREE_AT_ONCE)) {
        if (s == 0u && tid == 0u) ab.info[INFO_AHEAD] -= 1u;
        return;
    }
    if (tid < 2u * TREE_MAX_SEGMENTS) s_hi[tid] = room == TREE_NO_ROOM || tid >= 2u * tb.S ? 0u : my_hi;
    if (tid == 0u) s_state = 0u;
    const uint32_t per = min((count + tb.S - 1u) / tb.S, TREE_LAYERS), m = room == TREE_NO_ROOM ? 0u : min(per, count - min(s * per, count));
    // What a sum of the layers' errors in any order may differ from another: L roundings of at most half a unit each, of a
    // sum of at most the largest errors' sum; both sums, on both sides, and twice that.
    double abs_tot = 0.0;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) largest += __shfl_xor(largest, d, 64);
    if (lane == 0u) sd[wave] = largest;
    __syncthreads();
#pragma unroll
    for (uint32_t w = 0; w < WAVES; ++w) abs_tot += sd[w];
    const double margin = abs_tot * ((double)(L + 8u) * 0x1p-50);
    bool unsure = !(abs_tot < 1e300);
    if (NODES) {
#pragma unroll
        for (uint32_t lev = 0; lev < PATH_LEVELS; ++lev) {
            if (lev >= levels) continue;
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) {
                const uint32_t c = tid + (q & 1u) * NT;
                stage[(2u * lev + (q >> 1)) * 1024u + c] = c <= s_hi[2u * node_at(lev) + (q >> 1)] ? v[lev][q] : DP_INF;
            }
        }
    }
#pragma unroll
    for (uint32_t q = 0; q < LR; ++q) {
        const uint32_t r = wave + q * WAVES;
        const bool in = r < m && entry[q].w != 0xFFFFFFFFu;
        rec_e[r][lane] = in ? entry[q].e : DP_INF;
        rec_w[r][lane] = in ? entry[q].w : 0xFFFFFFFFu;
        rec_place[r][lane] = entry[q].place; rec_K[r][lane] = entry[q].K;
        const uint64_t near = ballot(in && entry[q].before <= entry[q].e + margin);     // (NaN for a single)
        if (lane == 0u) rec_near[r] = near;
    }
    // layers all of whose sizes cost the same: the best entry
    {
        uint32_t state = 0u;
#pragma unroll
        for (uint32_t q = 0; q < LT; ++q) {
            const uint32_t x = q * NT + tid, i = s * share + x;
            if (x >= share || i >= L) continue;
            if (bad[q]) state |= TREE_BAD;
            if (single[q].place == 0xFFFFFFFFu) continue;
            if (!(single[q].next > margin)) state |= TREE_UNSURE;
            if (single[q].before <= margin) state |= TREE_NEAR;
            tree_store(ab, tb, i, single[q].place, single[q].K);
        }
        if (state) atomicOr(&s_state, state);
    }
    // the least of total(y), y = lo .. hi, and the second least
    uint32_t turn = 0u;
    auto choose = [&](uint32_t lo, uint32_t hi, auto total) -> uint32_t {
        Two t{DP_INF, DP_INF, 0u};
        if (NODES) {
            for (uint32_t y = lo + lane; y <= hi; y += 64u) two_add(t, total(y), y);     // (every wave for itself)
            t = two_wave(t);
        } else {
            for (uint32_t y = lo + tid; y <= hi; y += NT) two_add(t, total(y), y);
            t = two_wave(t);
            turn ^= 1u;
            if (lane == 0u) s_two[turn][wave] = t;
            __syncthreads();
            t = Two{DP_INF, DP_INF, 0u};
            if (lane < WAVES) t = s_two[turn][lane];
            t = two_wave(t);
        }
        if (!(t.second > t.best + margin)) unsure = true;
        return t.at;
    };
    __syncthreads();
    if (m) {
        // ---- what this segment spends
        auto total = [&](uint32_t lev, uint32_t side, uint32_t c) {
            if (NODES) return stage[(2u * lev + side) * 1024u + c];
            return tb.vec[(size_t)(2u * node_at(lev) + side) * tb.pitch + c];
        };
        uint32_t x;
        if (levels == 0u) {
            x = choose(0u, min(s_hi[1], room), [&](uint32_t c) { return tb.vec[tb.pitch + c]; });
        } else {
            // the halves of the whole spend a and b, a + b <= room: the least of A[a] + (least B up to the rest)
            const uint32_t ha = s_hi[2], hb = s_hi[3];
            double b_of[PER], run = DP_INF;
#pragma unroll
            for (uint32_t q = 0; q < PER; ++q) {
                const uint32_t b = tid * PER + q;
                b_of[q] = b <= hb ? total(0u, 1u, b) : DP_INF;
                run = min_f64(run, b_of[q]);
            }
            const double incl = wave_scan_min_f64(run);
            double before = __shfl_up(incl, 1, 64);
            if (lane == 0u) before = DP_INF;
            if (lane == 63u) sd[8u + wave] = incl;
            __syncthreads();
            for (uint32_t w = 0; w < wave; ++w) before = min_f64(before, sd[8u + w]);
#pragma unroll
            for (uint32_t q = 0; q < PER; ++q) { before = min_f64(before, b_of[q]); least[tid * PER + q] = before; }
            __syncthreads();
            const uint32_t a = min(choose(0u, min(ha, room), [&](uint32_t y) { return total(0u, 0u, y) + least[min(room - y, hb)]; }), room);
            const uint32_t b = choose(0u, min(room - a, hb), [&](uint32_t y) { return total(0u, 1u, y); });
            x = (s >> (levels - 1u)) & 1u ? b : a;
            for (uint32_t lev = 1; lev < levels; ++lev) {
                const uint32_t k = 2u * node_at(lev), ga = s_hi[k], gb = s_hi[k + 1u];
                const uint32_t y = min(choose(x > gb ? x - gb : 0u, min(ga, x), [&](uint32_t c) { return total(lev, 0u, c) + total(lev, 1u, x - c); }), x);
                x = (s >> (levels - 1u - lev)) & 1u ? x - y : y;
            }
        }
        // ---- its layers, from the last one back
        uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
        double val = tb.vec[(size_t)(tb.S + s) * tb.pitch + min(at, s_hi[tb.S + s])];
        uint32_t mine = 0u;                                    // lane r: layer r's entry
        for (uint32_t t1 = m; t1 > 0u;) {
            const uint32_t cells = at + 1u, rows = min(t1, PATH_STAGE / cells), t0 = t1 - rows;
            __syncthreads();                                   // (the nodes' totals, or the rows before, are done with)
            // the rows that steps t0 .. t1 - 1 come from
            for (uint32_t r = wave; r < rows; r += WAVES) {
                const uint32_t p = max(t0 + r, 1u) - 1u;
                const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)my_row_hi, (int)p);
                const double* row = tb.rows + (size_t)(uint32_t)__builtin_amdgcn_readlane((int)my_layer, (int)p) * tb.pitch;
                for (uint32_t c0 = lane; c0 < cells; c0 += 512u) {
                    double from[8];
#pragma unroll
                    for (uint32_t q = 0; q < 8u; ++q) from[q] = c0 + 64u * q <= hi ? row[c0 + 64u * q] : DP_INF;
#pragma unroll
                    for (uint32_t q = 0; q < 8u; ++q) {
                        const uint32_t c = c0 + 64u * q;
                        if (c < cells) stage[r * cells + c] = t0 + r == 0u ? (c ? DP_INF : 0.0) : from[q];
                    }
                }
            }
            __syncthreads();
            if (wave == 0u) {
                uint32_t w = rec_w[t1 - 1u][lane];
                double e = rec_e[t1 - 1u][lane];
                for (uint32_t r = rows; r-- > 0u;) {
                    // (the layer before's entries are under way)
                    const uint32_t before = t0 + max(r, 1u) - 1u, w_next = rec_w[before][lane];
                    const double e_next = rec_e[before][lane];
                    const bool in = w <= at;
                    const double from = stage[r * cells + (in ? at - w : 0u)];
                    const double sum = from + e;
                    const uint64_t hit = ballot(in && sum == val), close = ballot(in && sum <= val + margin);
                    if (!hit || (close & (close - 1ull))) unsure = true;
                    const int k = hit ? (int)__builtin_ctzll(hit) : 0;
                    if (lane == t0 + r) mine = (uint32_t)k;
                    const uint32_t spent = (uint32_t)__builtin_amdgcn_readlane((int)w, k);
                    at = spent <= at ? at - spent : 0u;
                    val = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(from), k), __builtin_amdgcn_readlane(__double2loint(from), k));
                    w = w_next; e = e_next;
                }
                if (t0 == 0u && lane < m) {
                    tree_store(ab, tb, my_layer, rec_place[lane][mine], rec_K[lane][mine]);
                    if ((rec_near[lane] >> mine) & 1ull) atomicOr(&s_state, (uint32_t)TREE_NEAR);
                }
                if (lane == 0u) { s_x = at; sd[0] = val; }
            }
            t1 = t0;
            if (t1) {
                __syncthreads();
                at = s_x; val = sd[0];
            }
        }
    }
    // ---- the segment that is through last goes on (what the others stored beyond the caches is there)
    if (unsure && lane == 0u) atomicOr(&s_state, (uint32_t)TREE_UNSURE);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0u) {
        if (s_state) {
            atomicOr(&tb.head[2], s_state);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        s_last = atomicAdd(&tb.head[1], 1u) + 1u == gridDim.x ? 1u : 0u;
    }
    __syncthreads();
    if (!s_last) return;
    const uint32_t state = __hip_atomic_load(&tb.head[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t K[LT], entry_at[LT];                              // of layers LT tid + q
    int32_t j[LT];
#pragma unroll
    for (uint32_t q = 0; q < LT; ++q) {
        const uint32_t i = min(LT * tid + q, L - 1u);
        K[q] = (uint32_t)__hip_atomic_load(&ab.K_out[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        j[q] = __hip_atomic_load(&ab.j_out[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        entry_at[q] = __hip_atomic_load(&tb.at[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const int32_t st = state & TREE_BAD ? err_nonfinite : room == TREE_NO_ROOM ? err_infeasible : 0;
    const bool chain = st == 0 && (state & TREE_UNSURE);
    if (tid == 0u) {
        tb.head[3] = chain ? 1u : 0u;
        alloc_decided(ab, chain);
        if (!chain && st == 0 && (state & TREE_NEAR)) ab.info[INFO_HOW] = HOW_FROM_LEFT;
        if (!chain) *ab.status = st;
    }
    if (chain) {
        for (uint32_t r = wave; r <= L; r += WAVES) dp_fill_row(ab, tb.rows, tb.pitch, 0u, r, lane, 64u);
        if (tid < 4u) ab.flags[tid] = tid == 1u ? ab.first_ticket : 0u;
        return;
    }
    if (st != 0) {
        for (uint32_t i = tid; i < L; i += NT) { ab.j_out[i] = 0; ab.K_out[i] = 0; }
        for (uint32_t i = tid; i <= L; i += NT) ab.offsets_out[i] = 0;
        step_lookup(sl, NT);
        return;
    }
    // Of a run of equal costs the chain names the lowest member whose rounded total is the last one's: where one of another error is
    // that near, the totals from the left are formed.
    if (state & TREE_NEAR) {
        // Bound by memory round trips, then by one thread's additions: the member's error, its neighbour's below and the run's first
        // member are asked for together, and the terms come eight at a time.  (us, one after another throughout, and so: ResNet-50's
        // 161 layers 3.8 and 3.1, with a wide link 6.5 and 3.9, ResNet-18's 62 3.4 and 2.0.)
        constexpr uint32_t AT_A_TIME = 8u;
        double *term = stage, *total = stage + TREE_MAX_L + 2u * AT_A_TIME;
        static_assert(PATH_STAGE >= 2u * (TREE_MAX_L + 2u * AT_A_TIME), "the path's totals fit");
        double below[LT];
        uint32_t K_below[LT], first[LT];
        if (tid < 2u * AT_A_TIME) term[L + tid] = 0.0;
#pragma unroll
        for (uint32_t q = 0; q < LT; ++q) {
            const uint32_t i = min(LT * tid + q, L - 1u);
            const size_t row = (size_t)i * ab.J;
            const uint32_t own = min((uint32_t)j[q], ab.J - 1u), under = max(own, 1u) - 1u;
            const double e = ab.E[row + own];
            below[q] = ab.E[row + under]; K_below[q] = ab.Kout[row + under];
            first[q] = dl.jj[row + min(entry_at[q], ab.J - 1u)] & 0xFFu;
            if (LT * tid + q < L) term[i] = e;
        }
        __syncthreads();
        if (tid == 0u) {
            double run = 0.0, t[AT_A_TIME], ahead[AT_A_TIME];
#pragma unroll
            for (uint32_t u = 0; u < AT_A_TIME; ++u) t[u] = term[u];
            for (uint32_t i = 0; i < L; i += AT_A_TIME) {
#pragma unroll
                for (uint32_t u = 0; u < AT_A_TIME; ++u) ahead[u] = term[i + AT_A_TIME + u];
#pragma unroll
                for (uint32_t u = 0; u < AT_A_TIME; ++u) { total[i + u] = run; run += t[u]; }
#pragma unroll
                for (uint32_t u = 0; u < AT_A_TIME; ++u) t[u] = ahead[u];
            }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < LT; ++q) {
            const uint32_t i = LT * tid + q;
            if (i >= L) continue;
            const double from = total[i], to = from + term[i];
            uint32_t low = (uint32_t)j[q];
            if (low <= first[q] || from + below[q] != to) continue;
            K[q] = K_below[q];
            for (--low; low > first[q] && from + ab.E[(size_t)i * ab.J + low - 1u] == to;) K[q] = ab.Kout[(size_t)i * ab.J + --low];
            j[q] = (int32_t)low;
        }
    }
    // offsets: the sizes' low 22 bits and the rest of them are summed up apart (1024 of either stay within 32 bits)
    static_assert(TREE_MAX_L <= 1024, "of 22 bits");
    uint32_t lo = 0u, up = 0u;
#pragma unroll
    for (uint32_t q = 0; q < LT; ++q)
        if (LT * tid + q < L) { lo += K[q] & 0x3FFFFFu; up += K[q] >> 22; }
    const uint32_t lo_in = wave_scan_add_u32(lo), up_in = wave_scan_add_u32(up);
    if (lane == 63u) { su[0][wave] = lo_in; su[1][wave] = up_in; }
    __syncthreads();
    uint32_t lo_at = lo_in - lo, up_at = up_in - up;
    for (uint32_t w = 0; w < wave; ++w) { lo_at += su[0][w]; up_at += su[1][w]; }
    unsigned long long off = (unsigned long long)lo_at + ((unsigned long long)up_at << 22);
#pragma unroll
    for (uint32_t q = 0; q < LT; ++q) {
        const uint32_t i = LT * tid + q;
        if (i >= L) continue;
        ab.offsets_out[i] = off; ab.K_out[i] = K[q]; ab.j_out[i] = j[q];         // (stored again: the look-up reads them through the caches)
        off += K[q];
        if (i == L - 1u) ab.offsets_out[L] = off;
    }
    step_lookup(sl, NT);
}

}  // namespace kimad
