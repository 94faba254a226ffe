// C ABI of the library: argument checks, workspace layout, kernel launches.
// Declarations and the contract of every entry point are in include/kimad.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <numeric>
#include <type_traits>
#include <vector>

#include "../../include/kimad.h"
#include "common.h"
#include "shares.h"
#include "k_profile.h"
#include "k_fused.h"
#include "k_compress.h"
#include "k_alloc.h"
#include "k_alloc_chain.h"
#include "k_alloc_band.h"
#include "k_alloc_tree.h"
#include "k_alloc_halves.h"
#include "k_server.h"
#include "k_selftest.h"

static_assert(kimad::KIMAD_MAX_J_CONST == KIMAD_MAX_J, "J limit mismatch");

namespace {

using namespace kimad;

constexpr uint64_t ALIGN = 256;
// A table entry is accepted from the two histogram levels when its rigorous error bound is
// below this fraction of the entry; otherwise the exact last-digit pass recomputes it.
constexpr double CERT_TOL = 4e-6;
constexpr double SLOT_WIDEN = 1.2e-7;      // half width (relative) of the midpoint form of a single-pass slot's squares

inline uint64_t align_up(uint64_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }

// Byte offsets of every array inside the workspace.
struct Layout {
    uint32_t L = 0, J = 0, B = 0, S = 0;
    uint32_t tile_elems = 0, ntiles = 0, nchunks = 0, nswg = 0, ncblk = 0;
    uint64_t dp_cells = 0, tmp_cap = 0, sum_kmax = 0;
    // static tables
    uint64_t layers, ktab, tile_layer, chunk_big, chunk_first, big_layer, small_layer;
    // zeroed before every profile
    uint64_t swg_layer, swg_first, state, lutc;
    uint64_t fresh = 0, hprev = 0, gprev = 0;
    uint64_t zero1_begin, cnt1, sq1, cnt2, sq2, diag, layer_flag, shist, ghist, cursor, spill_over, tiles_done, zero1_end;
    uint64_t cprev = 0;
    uint64_t big_tmp0, parts, part_head, shares, reduce_layers, zero1_mid;
    uint32_t main_wgs = 0, nparts = 0, nsplit = 0;
    uint64_t pool_prefix, pool_big, pool_t0, pool_cnt, pool_hist, tgt_unsel, tgt_base;
    uint32_t pool_cap = 1;
    uint64_t lut1, nslots, slot_bin, slot_cnt, slot_sq;
    uint64_t tgt_slot, tgt_r, tgt_above1, tgt_below, sel_prefix, sel_above, sel_amb;
    // compress
    uint64_t ksel, sel, zero2_begin, hist3, zero2_end, tau, quota, cblk_big;
    uint64_t rec_start, rec_cnt, rec_amb, c_gt, c_eq, o_base, o_allow;
    uint64_t tmp_x, tmp_i;
    // allocation
    uint64_t ncompact;
    uint64_t row0, row1, choice, dp_flags, dl_wall, dl_w, dl_jj, dl_e, dl_n, dl_bad, rows_g;
    uint64_t dense_E, dense_Kcost, dense_Kout;
    uint64_t band_lo, band_hi, band_info, band_live, hull_e, hull_w, hull_n, hull_abs;
    uint64_t half_order;
    uint64_t tree_vec, tree_hi, tree_entry, tree_layer, tree_row_hi, tree_single, tree_at, tree_head;
    uint64_t rstride = 0;            // cells per stored DP row (LDS-resident recurrence only)
    uint64_t total = 0, least = 0;   // least: without the rows that only k_dp_chain_long takes
};

struct HostLayer {
    uint32_t n, mis, hvec;
    int32_t big;
    uint32_t tile0, ntiles, chunk0, nchunks;
    uint32_t sstride, sgroups, swg0, nswg;   // sampling: stride in chunks, sampled groups, workgroups
    uint32_t cblk0, ncblk;                   // blocks of 1024 chunks
    uint64_t tmp0;                           // region start in the candidate buffer
    uint32_t tmp_cap;                        // entries of the region
};

// Rows too long for LDS: pitch of a stored row, and whether the workspace holds one per layer (k_dp_chain_long); else the
// layers are launched one by one on two rows.  (The line is the memory: k_dp_chain_long was faster at every length tried.)
constexpr uint64_t CHAIN_LONG_BYTES = 256ull << 20;
inline uint64_t chain_long_pitch(uint64_t cells) { return (CHAIN_PAD + cells + 63ull) & ~63ull; }
inline bool chain_long_fits(uint64_t L, uint64_t cells) {
    return cells > DP_ROW_MAX && 8ull * (L + 1) * chain_long_pitch(cells) <= CHAIN_LONG_BYTES;
}

// Rows that fit LDS go by the tree of segments (k_alloc_tree.h) from so many layers on: below, the chain's few steps, or for longer rows
// the band, take less than the tree's launches.  us of all launches of the allocation, chain and tree, layers of 5 and of 64 ratios:
//   256 cells  60 layers 31 and 32, 33 and 34; 64 layers 32 and 32, 35 and 33; 74 layers 34 and 33, 37 and 34
//   384        60 32 and 33, 34 and 35; 64 33 and 33, 36 and 35
//   500        60 33 and 34, 35 and 36; 64 34 and 34, 36 and 36; 74 37 and 35, 39 and 38; 161 60 and 40, 63 and 40
//   512        60 33 and 34, 35 and 36
//   600        60 34 and 34, 41 and 38; 700 cells 38 and 35, 41 and 39
//   1000       60 41 and 37, 48 and 41 (21 of 64 31 and 41, 53 of 16 40 and 43); 161 75 and 43, 78 and 47; 700 of 33 230 and 64
//   1025       60 46 and 35, 53 and 43; 161 85 and 42, 87 and 49
//   1536       60 51 and 38, 62 and 47; 300 145 and 49, 151 and 54
// and from BAND_AUTO_CELLS on the better of chain and band, layers of 2, 16 and 64 ratios:
//   1537       24 36 and 31, 37 and 37, 40 and 48 (band 58); 40 44 and 34, 45 and 38, 50 and 49; 161 91 and 45, 92 and 47, 98 and 54
//   4097       24 56 and 38, 56 and 46, 61 and 73 (band 69); 40 78 and 45, 75 and 51, 78 and 68; 161 216 and 66, 170 and 69, 193 and 84
// Where rounding may decide, the chain comes behind it, and behind ties in a row at once: chain or band alone, both, and the chain at once,
// 148 layers of 16 and of 64 ratios: 1000 cells 72, 118, 84 and 107, 154, 119; 4097 cells 183, 302, 230 and 223, 352, 284.
constexpr uint32_t TREE_MIN_L = 24, TREE_MIN_L_SHORT = 60;       // (rows of fewer than BAND_AUTO_CELLS cells: the latter;
constexpr uint32_t TREE_MIN_L_SHORTEST = 64, TREE_SHORTEST = 576;          //  of fewer than TREE_SHORTEST cells: this)
// Segments of at most this many layers: a segment's layers are one after another, a level of the tree is a launch.  (us with 3, 6 and
// 12: rows of 1000 cells, 148 layers of 64 ratios 60, 56, 56, 218 of 64 65, 65, 74, 62 of 50 41, 41, 46.  Of 4097 cells, whose
// levels cost more, 148 of 64 172, 138, 117, 161 of 64 74, 73, 78.)
constexpr uint32_t TREE_FEW = 6, TREE_FEW_LONG = 12;
// A join of rows of more than 1024 cells takes 64 costs a workgroup where that makes a workgroup a compute unit and a few more, else 32.
// (us of all launches of the allocation with 64 costs from 0, 100, 200, 300 and 600 such workgroups on, and never: 96 layers of 16 ratios, a
// join of two and one of four nodes, 2048 cells 50, 48, 47, 47, 47, 47, 4097 70, 69, 66, 64, 64, 64; 190 layers, eight nodes too, 2048 55, 54,
// 52, 52, 52, 52, 4097 75, 75, 72, 73, 75, 74; 760, sixteen and 32 too, 2560 65, 64, 63, 64, 63, 66, 3600 76, 76, 74, 73, 74, 78.)
constexpr uint32_t JOIN_WIDE_WGS = 300;
inline bool tree_takes(uint64_t L, uint64_t J) { return L >= TREE_MIN_L && L <= TREE_MAX_L && J > 1; }
inline uint32_t tree_segments(uint64_t layers, uint32_t few) {
    uint32_t s = 1;
    while (s < TREE_MAX_SEGMENTS && (uint64_t)s * few < layers) s <<= 1;
    return s;
}

// Rows beyond LDS go by halves (k_alloc_halves.h) from so many layers on; fewer do not pay for the three launches more, and the three that
// leave at once, and nor do some more whose steps are short, of up to sixteen candidates over shorter rows.  us of all launches of the
// allocation, one chain and halves: 62 layers of 32 candidates and 58 thousand cells 174 and 122, of 131 thousand 262 and 167, 161 of 64 and
// 13 thousand 404 and 260; 16 layers of 17 candidates and 4300 cells 42 and 42, of 64 52 and 49; 16 of 16 and 4300 35 and 39, 13 thousand
// 38 and 40, 20 thousand 45 and 43, 42 thousand 59 and 50; 20 of 16 and 4300 39 and 42, 13 thousand 44 and 44; 24 45 and 45, 49 and 46, 30 52 and
// 50, 57 and 53; 8 of 5 and 9 thousand 26 and 33.  Where rounding may decide, one chain comes
// behind them (k_dp_refill).
constexpr uint32_t HALVES_MIN_L = 16, HALVES_MIN_L_SHORT = 24;          // (the latter: up to HALVES_FEW_J ratios, fewer than HALVES_LONG cells)
constexpr uint32_t HALVES_FEW_J = 16, HALVES_LONG = 16384;

uint32_t pick_tile_elems(uint64_t d_big) {
    // aim at >= 8 tiles per compute unit on large inputs, keep tiles within the 16-bit LDS counters
    uint64_t t = 32768;
    while (t > 2048 && d_big / t < 256ull * 8ull) t >>= 1;
    return (uint32_t)t;
}

uint32_t grid_size_K(double r, uint64_t n) {
    double k = std::ceil(r * (double)n);
    if (k < 1.0) k = 1.0;
    if (k > (double)n) k = (double)n;
    return (uint32_t)k;
}

// Shapes only: misalignment is taken as the worst case (3) so that the layout does not depend on
// pointer values and kimad_workspace_bytes can be called before the tensors exist.
// Workgroups of the streaming pass: one per compute unit of the current device (256 if no device
// answers, as when only the workspace size is asked for on a machine without one), at most 1024,
// and at most cfg.max_workgroups.
uint32_t stream_workgroups(const kimad_config_t& cfg) {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) {
        (void)hipGetLastError();
        cus = 256;
    }
    uint32_t w = (uint32_t)std::min(cus, 1024);
    if (cfg.max_workgroups) w = std::min(w, cfg.max_workgroups);
    return w;
}

// A workgroup of the streaming pass starts a new histogram (a part) at every layer boundary of its share and, where a count may
// fill up, no earlier than after PK_MAX_CHUNKS chunks.
struct PartTables {
    std::vector<MainShare> shares;               // one more than there are workgroups
    std::vector<uint32_t> big_part0, big_nparts;
    // the layers in the order in which their parts are summed up: those whose blocks take a workgroup each (split) first,
    // which take longest
    std::vector<ReduceLayer> reduce_layers() const {
        std::vector<ReduceLayer> layers;
        for (int split = 1; split >= 0; --split)
            for (uint32_t b = 0; b < big_nparts.size(); ++b)
                if ((big_nparts[b] > REDUCE_WAVE_PARTS) == (split != 0)) layers.push_back({b, big_part0[b], big_nparts[b], 0u});
        return layers;
    }
    uint32_t nsplit() const {
        return (uint32_t)std::count_if(big_nparts.begin(), big_nparts.end(), [](uint32_t n) { return n > REDUCE_WAVE_PARTS; });
    }
};
// Returns the number of parts.
uint32_t plan_parts(const std::vector<HostLayer>& hl, uint32_t B, uint32_t nchunks, uint32_t wgs, PartTables& out) {
    std::vector<uint32_t> ends(B), li(B);
    for (uint32_t i = 0; i < hl.size(); ++i)
        if (hl[i].big >= 0) { ends[hl[i].big] = hl[i].chunk0 + hl[i].nchunks; li[hl[i].big] = i; }
    std::vector<uint32_t> first = plan_shares(ends, wgs);
    first.push_back(nchunks);
    out.shares.clear(); out.big_part0.assign(B, 0); out.big_nparts.assign(B, 0);
    uint32_t part = 0, b = 0;
    for (size_t w = 0; w + 1 < first.size(); ++w) {
        uint32_t cur = first[w];
        if (cur == ends[b]) ++b;
        out.shares.push_back({cur, part, b, li[b]});
        while (cur < first[w + 1]) {
            if (cur == ends[b]) ++b;
            if (out.big_nparts[b]++ == 0) out.big_part0[b] = part;
            ++part;
            cur = std::min<uint32_t>(std::min(first[w + 1], ends[b]), cur + PK_MAX_CHUNKS);
        }
    }
    out.shares.push_back({nchunks, part, 0u, 0u});
    return part;
}

int make_layout(const uint64_t* n, uint32_t L, uint32_t J, const kimad_config_t& cfg, Layout& lo,
                std::vector<HostLayer>* hl_out, PartTables* parts_out = nullptr) {
    std::vector<HostLayer> hl_local;
    std::vector<HostLayer>* hl = hl_out ? hl_out : &hl_local;
    if (!n || L == 0 || L > 65535 || J == 0 || J > KIMAD_MAX_J) return KIMAD_ERR_INVALID_ARG;
    lo.L = L; lo.J = J;
    uint64_t d_big = 0, d_all = 0;
    uint32_t B = 0, S = 0;
    for (uint32_t i = 0; i < L; ++i) {
        if (n[i] == 0 || n[i] > KIMAD_MAX_N) return KIMAD_ERR_INVALID_ARG;
        d_all += n[i];
        if (n[i] > SMALL_MAX) { d_big += n[i]; ++B; } else ++S;
    }
    lo.B = B; lo.S = S;
    lo.tile_elems = pick_tile_elems(d_big);
    uint64_t nt = 0, nc = 0, tmp_run = 0;
    uint32_t nsw = 0, ncblk = 0;
    hl->resize(L);
    int32_t bi = 0;
    for (uint32_t i = 0; i < L; ++i) {
        HostLayer h{};
        h.n = (uint32_t)n[i];
        h.big = -1;
        if (n[i] > SMALL_MAX) {
            const uint64_t span = n[i] + 3;
            h.big = bi++;
            h.tile0 = (uint32_t)nt; h.ntiles = (uint32_t)((span + lo.tile_elems - 1) / lo.tile_elems);
            h.chunk0 = (uint32_t)nc; h.nchunks = (uint32_t)((span + CHUNK - 1) / CHUNK);
            nt += h.ntiles; nc += h.nchunks;
            // sample one chunk in every `sstride`, keeping at least ~64 sampled chunks per layer
            h.sstride = std::max<uint32_t>(1, std::min<uint32_t>(16, h.nchunks / 64));
            h.sgroups = (h.nchunks + h.sstride - 1) / h.sstride;
            h.swg0 = nsw; h.nswg = (h.sgroups + SAMPLE_GROUPS_PER_WG - 1) / SAMPLE_GROUPS_PER_WG;
            nsw += h.nswg;
            h.tmp0 = region_start(h.chunk0, (uint32_t)h.big); h.tmp_cap = h.nchunks * REGION_PER_CHUNK + REGION_SLACK;
            tmp_run = h.tmp0 + h.tmp_cap;                 // the regions follow one another: region_start says where
            h.cblk0 = ncblk; h.ncblk = (h.nchunks + CBLOCK - 1) / CBLOCK; ncblk += h.ncblk;
        }
        (*hl)[i] = h;
    }
    lo.nswg = nsw;
    lo.ncblk = ncblk;
    if (nt > 0x7FFFFFFFull || nc > 0xFFFFFFFFull) return KIMAD_ERR_INVALID_ARG;
    lo.ntiles = (uint32_t)nt; lo.nchunks = (uint32_t)nc;
    lo.sum_kmax = d_all;                                  // the last grid ratio may be 1
    const uint32_t pair = cfg.pair_bytes ? cfg.pair_bytes : 8u;
    if (cfg.cost_units_D) {
        lo.dp_cells = std::min<uint64_t>(cfg.cost_units_D, d_all) + 1;
    } else {
        uint64_t pmax = cfg.max_budget_bytes ? cfg.max_budget_bytes / pair : d_all;
        lo.dp_cells = std::min<uint64_t>(pmax, d_all) + 1;
    }
    // (the winners' table of the allocation is L rows of dp_cells bytes: with the exact cost axis and no
    // budget limit that is L * d bytes, 18 GB for a 124M-element model: refused rather than asked of the caller)
    if ((uint64_t)L * align_up(lo.dp_cells) > (4ull << 30)) return KIMAD_ERR_TABLES_TOO_LARGE;
    lo.tmp_cap = tmp_run;                                 // one region per tiled layer
    PartTables parts_local;
    PartTables& parts = parts_out ? *parts_out : parts_local;
    lo.nparts = plan_parts(*hl, B, lo.nchunks, stream_workgroups(cfg), parts);
    lo.main_wgs = (uint32_t)parts.shares.size() - 1u;
    lo.nsplit = parts.nsplit();

    uint64_t off = 0;
    auto take = [&](uint64_t bytes) { uint64_t o = off; off = align_up(off + bytes); return o; };
    const uint64_t LJ = (uint64_t)L * J;
    lo.layers = take(sizeof(LayerDesc) * (uint64_t)L);
    lo.ktab = take(4 * LJ);
    lo.tile_layer = take(4ull * (nt ? nt : 1));
    lo.chunk_big = take(4ull * (nc ? nc : 1));
    lo.chunk_first = take(4ull * (nc ? nc : 1));
    lo.big_layer = take(4ull * (B + 1ull));               // (k_main reads a layer ahead)
    lo.big_tmp0 = take(8ull * (B ? B : 1));
    lo.shares = take(sizeof(MainShare) * parts.shares.size());
    lo.reduce_layers = take(sizeof(ReduceLayer) * (uint64_t)(B ? B : 1));
    // (the exact pass's pool of last-digit histograms lives in the same memory: the parts are dead once
    // k_reduce_parts has run, and a pool entry is cleared by the workgroup that takes it)
    lo.pool_cap = (uint32_t)std::min<uint64_t>(std::max<uint64_t>((uint64_t)B * J, 1), POOL_LIMIT);
    lo.parts = take(std::max<uint64_t>(8ull * PART_STRIDE * (lo.nparts ? lo.nparts : 1), 4ull * lo.pool_cap * D3_BINS));
    lo.pool_hist = lo.parts;
    lo.part_head = take(4ull * PART_HEAD * lo.nparts);
    lo.small_layer = take(4ull * (S ? S : 1));
    lo.swg_layer = take(4ull * (nsw ? nsw : 1));
    lo.swg_first = take(4ull * (nsw ? nsw : 1));
    lo.state = take(sizeof(LayerState) * (uint64_t)(B ? B : 1));
    lo.lutc = take(1ull * B * D1_BINS);
    lo.zero1_begin = off;
    lo.cnt1 = take(4ull * B * D1_BINS);
    lo.sq1 = take(8ull * B * D1_BINS);
    lo.cnt2 = take(4ull * B * SLOT_STRIDE * D2_BINS);
    lo.sq2 = take(8ull * B * SLOT_STRIDE * D2_BINS);
    lo.zero1_mid = off;                                   // the single-pass profile writes the tables above whole
    lo.diag = take(16);
    lo.fresh = take(16);
    lo.layer_flag = take(4ull * (B ? B : 1));
    lo.shist = take(4ull * B * D1_BINS);
    lo.ghist = take(8ull * D1_BINS);
    lo.cursor = take(4ull * (B ? B : 1));
    lo.spill_over = take(4ull * (B ? B : 1));
    lo.tiles_done = take(4ull * (B ? B : 1));
    lo.rec_cnt = take(4ull * (nc ? nc : 1));              // chunk records start out as "nothing spilled"
    lo.zero1_end = off;
    lo.hprev = take(4ull * B * D1_BINS);
    lo.gprev = take(8ull * D1_BINS);
    lo.pool_prefix = take(4ull * lo.pool_cap);
    lo.pool_big = take(4ull * lo.pool_cap);
    lo.pool_t0 = take(4ull * lo.pool_cap);
    lo.pool_cnt = take(4ull * lo.pool_cap);
    lo.tgt_unsel = take(4 * LJ);
    lo.tgt_base = take(8 * LJ);
    lo.lut1 = take(1ull * B * D1_BINS);
    lo.nslots = take(4ull * (B ? B : 1));
    lo.slot_cnt = take(4ull * (B ? B : 1) * SLOT_STRIDE);
    lo.slot_sq = take(8ull * (B ? B : 1) * SLOT_STRIDE);
    lo.slot_bin = take(4ull * B * SLOT_STRIDE);
    lo.tgt_slot = take(4 * LJ);
    lo.tgt_r = take(4 * LJ);
    lo.tgt_above1 = take(4 * LJ);
    lo.tgt_below = take(8 * LJ);
    lo.sel_prefix = take(4 * LJ);
    lo.sel_above = take(4 * LJ);
    lo.sel_amb = take(4 * LJ);
    lo.ksel = take(4ull * L);
    lo.sel = take(sizeof(SelRec) * (uint64_t)(B ? B : 1));
    lo.zero2_begin = off;
    lo.hist3 = take(4ull * B * D3_BINS);
    lo.zero2_end = off;
    lo.cblk_big = take(4ull * (ncblk ? ncblk : 1));
    lo.tau = take(4ull * (B ? B : 1));
    lo.quota = take(4ull * (B ? B : 1));
    const uint64_t ncb = 4ull * (nc ? nc : 1);
    lo.rec_start = take(ncb); lo.rec_amb = take(ncb);
    lo.c_gt = take(ncb); lo.c_eq = take(ncb); lo.o_base = take(ncb); lo.o_allow = take(ncb);
    lo.tmp_x = take(4 * lo.tmp_cap); lo.tmp_i = take(2 * lo.tmp_cap);
    lo.row0 = take(8 * lo.dp_cells);
    lo.row1 = take(8 * lo.dp_cells);
    lo.choice = take((uint64_t)L * align_up(lo.dp_cells));
    lo.cprev = take(2ull * Pieces(L).count() * align_up(std::min<uint64_t>(lo.dp_cells, DP_ROW_MAX)));
    lo.dp_flags = take(4 * DP_FLAGS);
    lo.ncompact = take(16);
    lo.half_order = take(4ull * L);
    lo.dl_wall = take(4 * LJ); lo.dl_w = take(4 * LJ); lo.dl_jj = take(4 * LJ); lo.dl_e = take(16 * LJ); lo.dl_n = take(4ull * L);
    lo.dl_bad = take(4ull * L);
    lo.dense_E = take(8 * LJ); lo.dense_Kcost = take(4 * LJ); lo.dense_Kout = take(4 * LJ);
    lo.band_lo = take(4ull * (L + 1)); lo.band_hi = take(4ull * (L + 1));
    lo.band_info = take(4 * INFO_WORDS);
    lo.band_live = take(4ull * L);
    lo.hull_e = take(8 * LJ); lo.hull_w = take(4 * LJ); lo.hull_n = take(4ull * L); lo.hull_abs = take(8ull * L);
    {
        const uint64_t cells = std::min<uint64_t>(lo.dp_cells, DP_ROW_MAX);
        lo.rstride = 512ull * (cells <= 1024 ? 2 : cells <= 2048 ? 4 : cells <= 3072 ? 6 : 9);
    }
    if (tree_takes(L, J)) {
        const uint64_t S = tree_segments(L, TREE_FEW), slots = S * TREE_LAYERS;
        lo.tree_vec = take(16 * S * lo.rstride); lo.tree_hi = take(8 * S);
        lo.tree_entry = take(sizeof(TreeEntry) * 64 * slots); lo.tree_layer = take(4 * slots); lo.tree_row_hi = take(4 * slots);
        lo.tree_single = take(sizeof(TreeSingle) * (uint64_t)L); lo.tree_at = take(4ull * L);
        lo.tree_head = take(32);
    }
    // (last: a workspace that ends with the shorter rows is accepted too, see kimad_plan::all_rows)
    lo.rows_g = take(8ull * (L + 1) * lo.rstride);
    lo.least = lo.total = off;
    if (chain_long_fits(L, lo.dp_cells)) lo.total = std::max(lo.total, lo.rows_g + align_up(8ull * (L + 1) * chain_long_pitch(lo.dp_cells)));
    return KIMAD_OK;
}

kimad_config_t normalise(const kimad_config_t* cfg) {
    kimad_config_t c{};
    if (cfg) c = *cfg;
    if (c.pair_bytes == 0) c.pair_bytes = c.value_format == KIMAD_VALUES_F16 ? 6 : 8;
    return c;
}

// Pairs of one cost unit of an allocation that spends P pairs.
uint64_t cost_unit(const kimad_config_t& cfg, uint64_t P) {
    const uint64_t D = cfg.cost_units_D;
    return D == 0 || P <= D ? 1 : (P + D - 1) / D;
}

// Rows from this many cost cells on take the banded recurrence by themselves where the layers are too few for the tree.
constexpr uint64_t BAND_AUTO_CELLS = 1537;
// With few ratios the lists are short, and whole rows by many workgroups are cheaper than a band by one.
constexpr uint32_t WHOLE_ROWS_J = 7;
constexpr uint64_t WHOLE_ROWS_CELLS = 2048;
// From this many chunks in tiled layers on the candidates are stored nontemporally: what the pass writes no longer finds room
// in the 256 MB cache.  us of k_main with ordinary and with nontemporal stores: 480 K chunks and 1.1 % of the entries 702 and
// 709; 570 K and 4.6 % 954 and 924; 900 K and 4.6 % 1617 and 1477; 1.2 M and 1.1 % 1906 and 1807, 9 % 2593 and 2193.  Smaller
// sets lose by it (240 K chunks, 3 %: 370 and 383; 120 K, 1.1 %: 181 and 185), and the kernels that read the candidates too.
constexpr uint32_t STREAM_CANDIDATES_CHUNKS = 524288;
// Up to this many small layers share the launch of a kernel on the main stream; more of them, several to a compute unit in
// turn, go to the side stream beside what follows.  us in a shared launch and on the side stream, small layers of 768
// entries beside 20 tiled ones of 200 K: profile 67 and 80 with 64 of them, 72 and 80 with 512, 81 and 86 with 1024, 98 and 107
// with 2048; selection from scratch 97 and 109, 103 and 111, 115 and 119, 142 and 138.  Of 64 to 8192 entries beside 50 layers of
// 2 M: profile 227 and 235, 242 and 247, 257 and 265, 286 and 295; selection 425 and 429, 441 and 439, 448 and 443, 417 and
// 398.  The line is the selection's; the profile alone would go on sharing.
constexpr uint32_t SMALL_BESIDE = 512;
constexpr uint32_t FALLBACK_GRID = 1024;   // workgroups of a pass that usually has nothing to do
// The same for k_hist2, four times as many as fit: the layers to be recounted lie unevenly among the tiles.  (us with 512, 1024
// and 2048: 50 layers of the GPT-2-shaped set 323, 308, 293, 169 of the Llama-shaped set 2905, 2762, 2536, 53 of ResNet-50 78, 72,
// 72; with nothing to count 13.4 each.)
constexpr uint32_t RECOUNT_GRID = 2048;
// A selection from scratch takes the single pass from this many chunks in tiled layers on, if these hold this many each on
// average; below, its four more launches and its tables per layer cost more than the two reads of g and h it saves.
// A hundredth kept, single pass and two histogram passes with a compaction, us: 4 layers 81 and 71 at 1 M elements, 95 and
// 118 at 4 M; 60 layers 93 and 90 at 2.4 M, 101 and 133 at 6 M; one layer 98 and 93 at 2 M, 126 and 130 at 4 M, 134 and 196
// at 8 M.  2000 layers of 9000 to 16000 elements 10 to 20 % the other way, of 24000 644 and 670.  On the headline set at
// a hundredth 330 and 740, and 770 in a round whose every layer the prediction misses, as when all gradients are 64
// times the round before's.
constexpr uint32_t SINGLE_SELECT_CHUNKS = 3072;
constexpr uint32_t SINGLE_SELECT_PER_LAYER = 24;

__global__ __launch_bounds__(256) void k_zero16(uint4* p, uint64_t n16) {
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    for (uint64_t i = (uint64_t)blockIdx.x * 256u + threadIdx.x; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
}

__global__ __launch_bounds__(64) void k_fill_i32(int32_t* p, uint32_t n, int32_t v) {
    for (uint32_t i = threadIdx.x; i < n; i += 64u) p[i] = v;
}

// Entries of an ascending index list that fall into each layer's range of the flat buffer: two bisections a layer.
__global__ __launch_bounds__(256) void k_layer_counts(const uint32_t* __restrict__ idx, uint64_t pairs,
                                                      const uint64_t* __restrict__ layer_start, uint32_t L, uint64_t* counts) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= L) return;
    auto first_at_or_above = [&](uint64_t pos) {      // number of entries below position pos
        uint64_t lo = 0, hi = pairs;
        while (lo < hi) {
            const uint64_t mid = (lo + hi) >> 1;
            if ((uint64_t)idx[mid] < pos) lo = mid + 1; else hi = mid;
        }
        return lo;
    };
    counts[i] = first_at_or_above(layer_start[i + 1]) - first_at_or_above(layer_start[i]);
}

__global__ __launch_bounds__(256) void k_make_ksel(const uint64_t* K, const kimad::LayerDesc* layers, uint32_t L,
                                                   uint32_t* ksel) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i < L) {
        const uint64_t k = K[i];
        ksel[i] = k > layers[i].n ? layers[i].n : (uint32_t)k;
    }
}

}  // namespace

struct kimad_plan {
    Layout lo;
    kimad_config_t cfg;
    std::vector<HostLayer> hl;
    std::vector<uint32_t> ktab;      // host copy of K_ij
    std::vector<uint32_t> kmax;      // K_{i,J-1}
    double ratio0 = 0.0;             // the grid's smallest ratio
    char* ws = nullptr;
    bool all_rows = false;           // the workspace holds every row of an allocation beyond LDS (Layout::total)
    int device = 0;
    uint32_t main_wgs = 256;         // persistent workgroups of the fused pass (one per compute unit)
    kimad::ProfileBuffers pb;
    kimad::CompressBuffers cb;
    // optional per-kernel timing (events recorded after every launch)
    bool timing = false;
    std::vector<hipEvent_t> ev;
    std::vector<const char*> ev_name;
    uint32_t ev_n = 0;
    // The small layers (one workgroup each) do not depend on the tiled layers: where they are too many to share a
    // launch (SMALL_BESIDE), or the profile takes two full passes, their kernels run on a side stream, forked from and
    // joined back into the caller's stream with events, so that they overlap the short kernels of the tiled path.
    hipStream_t side = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    // The single-pass profile predicts from the exact histogram its previous run on this plan left behind, once
    // there is one (stream order makes it visible).
    bool hist_valid = false;
    ~kimad_plan() {
        for (hipEvent_t e : ev) (void)hipEventDestroy(e);
        if (ev_fork) (void)hipEventDestroy(ev_fork);
        if (ev_join) (void)hipEventDestroy(ev_join);
        if (side) (void)hipStreamDestroy(side);
    }
};

namespace {

template <typename T> T* at(kimad_plan* p, uint64_t off) { return reinterpret_cast<T*>(p->ws + off); }

constexpr uint32_t MAX_EVENTS = 1024;

// Stream for work that may overlap what follows on `s`: the side stream, made to wait for
// everything enqueued on `s` so far.  With per-kernel timing on (or if anything fails) it is `s`
// itself, i.e. plain in-order execution.
hipStream_t fork_side(kimad_plan* p, hipStream_t s) {
    if (p->timing || !p->side) return s;
    if (hipEventRecord(p->ev_fork, s) != hipSuccess) return s;
    if (hipStreamWaitEvent(p->side, p->ev_fork, 0) != hipSuccess) return s;
    return p->side;
}
int join_side(kimad_plan* p, hipStream_t s, hipStream_t used) {
    if (used == s) return KIMAD_OK;
    if (hipEventRecord(p->ev_join, used) != hipSuccess) return KIMAD_ERR_HIP;
    if (hipStreamWaitEvent(s, p->ev_join, 0) != hipSuccess) return KIMAD_ERR_HIP;
    return KIMAD_OK;
}

// With timing on, an event follows every launch; the interval between consecutive events is
// that kernel's duration on the stream.
void mark(kimad_plan* p, hipStream_t s, const char* name) {
    if (!p->timing || p->ev_n >= MAX_EVENTS) return;
    if (hipEventRecord(p->ev[p->ev_n], s) == hipSuccess) p->ev_name[p->ev_n++] = name;
}

#define KLAUNCH(p, s, name, kern, grid, block, ...)                    \
    do {                                                               \
        hipLaunchKernelGGL(kern, grid, block, 0, s, __VA_ARGS__);      \
        if (hipGetLastError() != hipSuccess) return KIMAD_ERR_HIP;     \
        mark(p, s, name);                                              \
    } while (0)

int zero_range(kimad_plan* p, uint64_t begin, uint64_t end, hipStream_t s) {
    const uint64_t n16 = (end - begin) / 16;
    if (n16 == 0) return KIMAD_OK;
    const uint32_t blocks = (uint32_t)std::min<uint64_t>((n16 + 255) / 256, 2048);
    KLAUNCH(p, s, "k_zero16", k_zero16, dim3(blocks), dim3(256), at<uint4>(p, begin), n16);
    return KIMAD_OK;
}

// Histogram passes + scans for a target table (the plan's grid, or one K per layer).
// mark_fresh: the targets are the plan's grid, i.e. this is kimad_profile (see ProfileBuffers::fresh).
// clear: the tables the passes add into (and the profile's "fresh" word) are cleared here; a caller that has
// already cleared them, before it let other kernels of the same call start on the side stream, passes false.
int run_select_passes(kimad_plan* p, const uint32_t* ktab_dev, uint32_t J, double* err_table, hipStream_t s,
                      uint32_t mark_fresh = 0u, bool clear = true) {
    const Layout& lo = p->lo;
    int rc = clear ? zero_range(p, lo.zero1_begin, lo.zero1_end, s) : KIMAD_OK;
    if (rc) return rc;
    if (lo.B) {
        KLAUNCH(p, s, "k_hist1", k_hist1, dim3(lo.ntiles), dim3(256), p->pb);
        KLAUNCH(p, s, "k_scan1", k_scan1, dim3(lo.B), dim3(256), p->pb, ktab_dev, J);
        const uint32_t group = hist2_group_tiles(lo.ntiles, lo.tile_elems);
        KLAUNCH(p, s, "k_hist2", k_hist2, dim3(lo.B + (lo.ntiles + group - 1) / group), dim3(HIST2_THREADS), p->pb, lo.B, lo.ntiles,
                (const uint32_t*)nullptr, 0u, ktab_dev, J, err_table, CERT_TOL, 0.0);
        // exact last-digit pass for the entries that the scan could not certify (usually none)
        if (err_table) KLAUNCH(p, s, "k_hist3p", k_hist3p, dim3(std::min<uint32_t>(lo.ntiles, FALLBACK_GRID)), dim3(HIST3_THREADS), p->pb, lo.ntiles, err_table, mark_fresh);
    }
    return KIMAD_OK;
}

// The small layers' profile as a launch of its own, on the side stream (more than SMALL_BESIDE of them: after the streaming
// pass is enqueued on `s`, so that they run beside the scans that follow it, which occupy a few dozen workgroups, and take no
// compute units from its persistent grid; or the two full passes, any number of them).
// *side gets the stream they were put on (to be joined by the caller).
int launch_small_profile(kimad_plan* p, double* err_table, hipStream_t s, hipStream_t* side,
                         const uint32_t* ktab_dev = nullptr, uint32_t J = 0) {
    const Layout& lo = p->lo;
    if (!lo.S) return KIMAD_OK;
    *side = fork_side(p, s);
    const uint32_t mark_fresh = ktab_dev ? 0u : 1u;       // other targets than the grid do not make a profile to reuse
    KLAUNCH(p, *side, "k_small_profile", k_small_profile, dim3(lo.S), dim3(SMALL_THREADS), p->pb,
            ktab_dev ? ktab_dev : (const uint32_t*)at<uint32_t>(p, lo.ktab), ktab_dev ? J : lo.J, err_table, mark_fresh);
    return KIMAD_OK;
}

// Single-pass profile: sample, predict, one streaming pass, candidate-fed digit-2 slots, and the
// classic recount only for layers whose prediction missed.
// ktab, J: the targets, the plan's grid or one size per layer; without an err_table only thresholds and candidates are
// wanted (a selection: no small layers, no certified errors).
int run_single_pass(kimad_plan* p, const uint32_t* ktab, uint32_t J, double* err_table, uint64_t budget_pairs, hipStream_t s,
                    hipStream_t* side) {
    const Layout& lo = p->lo;
    if (!lo.B) {
        int rc0 = zero_range(p, lo.zero1_mid, lo.zero1_end, s);
        if (rc0 || !err_table) return rc0;
        return launch_small_profile(p, err_table, s, side);
    }
    int rc = KIMAD_OK;
    const uint64_t unit = cost_unit(p->cfg, budget_pairs);
    const bool with_small = err_table && lo.S && lo.S <= SMALL_BESIDE;
    const dim3 grid(lo.B + (with_small ? lo.S : 0u)), block(with_small ? SMALL_THREADS : PREDICT_THREADS);
    if (p->hist_valid && !(p->cfg.flags & KIMAD_CFG_SAMPLE_ALWAYS)) {
        // prediction from the previous pass's exact histogram: no sampling pass, no clearing launch
        KLAUNCH(p, s, "k_predict", k_predict, grid, block, p->pb, lo.B, ktab, J, (unsigned long long)budget_pairs, (unsigned long long)unit,
                (const uint32_t*)p->pb.hprev, (const unsigned long long*)p->pb.gprev, 1u, err_table);
    } else {
        rc = zero_range(p, lo.zero1_mid, lo.zero1_end, s);   // the histogram tables are written whole by k_reduce_parts
        if (rc) return rc;
        KLAUNCH(p, s, "k_sample", k_sample, dim3(lo.nswg), dim3(SAMPLE_THREADS), p->pb);
        KLAUNCH(p, s, "k_predict", k_predict, grid, block, p->pb, lo.B, ktab, J, (unsigned long long)budget_pairs, (unsigned long long)unit,
                (const uint32_t*)p->pb.shist, (const unsigned long long*)p->pb.ghist, 0u, err_table);
    }
    p->hist_valid = true;
    if (lo.nchunks >= STREAM_CANDIDATES_CHUNKS) {
        KLAUNCH(p, s, "k_main", k_main<true>, dim3(p->main_wgs), dim3(FUSED_THREADS), p->pb);
    } else {
        KLAUNCH(p, s, "k_main", k_main<false>, dim3(p->main_wgs), dim3(FUSED_THREADS), p->pb);
    }
    KLAUNCH(p, s, "k_reduce_parts", k_reduce_parts, dim3(reduce_workgroups(lo.B, lo.nsplit)), dim3(256), p->pb, lo.nsplit);
    if (err_table && !with_small) {
        rc = launch_small_profile(p, err_table, s, side);
        if (rc) return rc;
    }
    KLAUNCH(p, s, "k_scan1x", k_scan1x, dim3(lo.B), dim3(SCAN1X_THREADS), p->pb, ktab, J);
    // a grid whose smallest ratio keeps a five-hundredth of a layer has no sparse slots (the two kernels' comments have both sides)
    if (err_table && p->ratio0 >= 1.0 / 512.0) {
        KLAUNCH(p, s, "k_hist2c", k_hist2c_dense, dim3((lo.nchunks + DENSE_CHUNKS - 1) / DENSE_CHUNKS), dim3(DENSE_THREADS), p->pb);
    } else {
        KLAUNCH(p, s, "k_hist2c", k_hist2c, dim3((lo.nchunks + 256u / SUB_HIST - 1) / (256u / SUB_HIST)), dim3(256), p->pb);
    }
    // the scan of every layer's slots, and a recount of the layers marked redo: a small grid, since there are none as a rule
    const uint32_t group = hist2_group_tiles(lo.ntiles, lo.tile_elems);
    KLAUNCH(p, s, "k_hist2", k_hist2, dim3(lo.B + std::min<uint32_t>((lo.ntiles + group - 1) / group, RECOUNT_GRID)), dim3(HIST2_THREADS), p->pb,
            lo.B, lo.ntiles, (const uint32_t*)(at<uint32_t>(p, lo.diag) + 3), 1u, ktab, J, err_table, CERT_TOL, SLOT_WIDEN);
    if (!err_table) return KIMAD_OK;
    KLAUNCH(p, s, "k_hist3p", k_hist3p, dim3(std::min<uint32_t>(lo.ntiles, FALLBACK_GRID)), dim3(HIST3_THREADS), p->pb, lo.ntiles, err_table, 1u);
    return KIMAD_OK;
}

// ---- allocation: the same kernels on two homes of their tables ----------------------------------
// Device memory the allocation's kernels work in besides their inputs and outputs.
struct AllocScratch {
    double* row0; double* row1;          // per-layer-launch path only
    uint8_t* choice; uint16_t* cprev;    // [L][pitch], [pieces][pitch]
    uint32_t* flags;                     // [DP_FLAGS]
    DpLists dl;
    BandBuffers band;
    double* dense_E; uint32_t* dense_Kcost; uint32_t* dense_Kout;   // [L][J] each: the tables as the dense fallback sees them
    double* rows_g;                      // [(L + 1)][rstride]
    uint32_t rstride;
    uint64_t max_cells;                  // longest row (capacity + 1) the tables hold
    bool all_rows;                       // rows_g holds all rows of that length (k_dp_chain_long)
    TreeBuffers tree;                    // (vec: null where there are none)
};

// Table memory for callers that cannot allocate (kimad_allocate_static): one array per device, inside the
// loaded code object.  Host code never passes the array's name to a kernel: it is a host-side stand-in,
// not a device address; the address of each device's copy is looked up once and kept.
constexpr uint64_t STATIC_SCRATCH_BYTES = 4096ull * 1024ull;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
unsigned char* g_scratch_ptr[MAX_DEVICES] = {};

// Address of the current device's copy of `scratch`, or nullptr on a HIP error.
unsigned char* static_scratch_of_current_device() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) { (void)hipGetLastError(); return nullptr; }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) { (void)hipGetLastError(); return nullptr; }
        g_scratch_ptr[dev] = static_cast<unsigned char*>(ptr);
    }
    return g_scratch_ptr[dev];
}

// The allocation's tables in the plan's workspace.
AllocScratch plan_scratch(kimad_plan* p) {
    const Layout& lo = p->lo;
    AllocScratch ws;
    ws.row0 = at<double>(p, lo.row0); ws.row1 = at<double>(p, lo.row1);
    ws.choice = at<uint8_t>(p, lo.choice); ws.cprev = at<uint16_t>(p, lo.cprev);
    ws.flags = at<uint32_t>(p, lo.dp_flags);
    ws.dl.wall = at<uint32_t>(p, lo.dl_wall); ws.dl.w = at<uint32_t>(p, lo.dl_w); ws.dl.jj = at<uint32_t>(p, lo.dl_jj);
    ws.dl.e = at<double>(p, lo.dl_e); ws.dl.n = at<uint32_t>(p, lo.dl_n); ws.dl.bad = at<uint32_t>(p, lo.dl_bad);
    ws.dense_E = at<double>(p, lo.dense_E); ws.dense_Kcost = at<uint32_t>(p, lo.dense_Kcost);
    ws.dense_Kout = at<uint32_t>(p, lo.dense_Kout);
    ws.band.lo = at<uint32_t>(p, lo.band_lo); ws.band.hi = at<uint32_t>(p, lo.band_hi);
    ws.band.info = at<uint32_t>(p, lo.band_info);
    ws.band.live = at<uint32_t>(p, lo.band_live);
    ws.dl.he = at<double>(p, lo.hull_e); ws.dl.hw = at<uint32_t>(p, lo.hull_w); ws.dl.hn = at<uint32_t>(p, lo.hull_n);
    ws.dl.habs = at<double>(p, lo.hull_abs);
    ws.rows_g = at<double>(p, lo.rows_g);
    ws.rstride = (uint32_t)lo.rstride;
    ws.max_cells = lo.dp_cells;
    ws.all_rows = p->all_rows && chain_long_fits(lo.L, lo.dp_cells);
    ws.tree = TreeBuffers{};
    if (tree_takes(lo.L, lo.J)) {
        TreeBuffers& t = ws.tree;
        t.vec = at<double>(p, lo.tree_vec); t.hi = at<uint32_t>(p, lo.tree_hi);
        t.entry = at<TreeEntry>(p, lo.tree_entry); t.layer = at<uint32_t>(p, lo.tree_layer); t.row_hi = at<uint32_t>(p, lo.tree_row_hi);
        t.single = at<TreeSingle>(p, lo.tree_single); t.at = at<uint32_t>(p, lo.tree_at);
        t.head = at<uint32_t>(p, lo.tree_head);
        t.rows = ws.rows_g; t.pitch = ws.rstride;
    }
    return ws;
}

int enqueue_allocate(kimad_plan* p, const AllocScratch& ws, const double* err_table, uint64_t budget_bytes,
                     int32_t* j_out, uint64_t* K_out, uint64_t* offsets_out, int32_t* status_out, hipStream_t s,
                     uint32_t polls = CHAIN_POLLS, uint32_t first_ticket = 0u, const StepLookup& sl = StepLookup{}) {
    const Layout& lo = p->lo;
    const uint64_t P = budget_bytes / p->cfg.pair_bytes;
    const uint64_t unit = cost_unit(p->cfg, P);
    uint64_t cap = P / unit;
    // Costs above the dearest allocation are unreachable (+inf for ever): cutting the rows there
    // changes no finite cell and so neither the least total nor the smallest cost attaining it.
    const bool dense = (p->cfg.flags & KIMAD_CFG_DENSE_FALLBACK) != 0;
    uint64_t wmax = 0;
    uint32_t choices = 0;                // layers whose sizes differ in cost
    for (uint32_t i = 0; i < lo.L; ++i) {
        uint64_t dearest = p->kmax[i], cheapest = p->ktab[(size_t)i * lo.J];
        const uint64_t n = p->hl[i].n, pb = p->cfg.pair_bytes;
        if (dense && cheapest * pb >= n * 4) cheapest = (n * 4 + pb - 1) / pb;
        if (dense && dearest * pb >= n * 4) dearest = (n * 4 + pb - 1) / pb;   // (costs ascend with j up to the break-even, and no grid point costs more than the dense size)
        wmax += (dearest + unit - 1) / unit;
        choices += (cheapest + unit - 1) / unit != (dearest + unit - 1) / unit;
    }
    if (cap > wmax) cap = wmax;
    if (cap + 1 > ws.max_cells) return KIMAD_ERR_INVALID_ARG;   // budget beyond what the tables were sized for

    AllocBuffers ab;
    ab.E = err_table; ab.Ktab = at<uint32_t>(p, lo.ktab); ab.Kout = ab.Ktab; ab.L = lo.L; ab.J = lo.J;
    ab.unit = unit; ab.cap = (uint32_t)cap;
    ab.row0 = ws.row0; ab.row1 = ws.row1;
    ab.choice = ws.choice; ab.cprev = ws.cprev; ab.stride = align_up(cap + 1);   // row pitch: <= align_up(max_cells)
    ab.j_out = j_out; ab.K_out = K_out; ab.offsets_out = offsets_out; ab.status = status_out;
    ab.flags = ws.flags; ab.polls = polls; ab.first_ticket = first_ticket; ab.info = ws.band.info;
    mark(p, s, "begin");
    if (dense) {
        KLAUNCH(p, s, "k_dense_view", k_dense_view, dim3((lo.L * lo.J + 255) / 256), dim3(256), err_table, ab.Ktab,
                (const LayerDesc*)at<LayerDesc>(p, lo.layers), lo.L, lo.J, p->cfg.pair_bytes, ws.dense_E, ws.dense_Kcost,
                ws.dense_Kout);
        ab.E = ws.dense_E; ab.Ktab = ws.dense_Kcost; ab.Kout = ws.dense_Kout;
    }
    if (cap + 1 <= DP_ROW_MAX) {
        const DpLists& dl = ws.dl;
        double* rows_g = ws.rows_g;
        const uint32_t rstride = ws.rstride;
        const bool long_rows = cap + 1 >= BAND_AUTO_CELLS && lo.J > 1 && !(lo.J <= WHOLE_ROWS_J && cap + 1 <= WHOLE_ROWS_CELLS);
        // (the withheld workgroup of the self-test is the chain's)
        const bool tree = ws.tree.vec && !(p->cfg.flags & (KIMAD_CFG_FULL_DP | KIMAD_CFG_BAND_DP)) && first_ticket == 0u &&
                          lo.L >= (cap + 1 >= BAND_AUTO_CELLS ? TREE_MIN_L : cap + 1 >= TREE_SHORTEST ? TREE_MIN_L_SHORT : TREE_MIN_L_SHORTEST);
        const bool band = lo.L <= BAND_MAX_L && !(p->cfg.flags & KIMAD_CFG_FULL_DP) &&
                          ((p->cfg.flags & KIMAD_CFG_BAND_DP) || (long_rows && lo.L < TREE_MIN_L));
        // (keepers of 16 cells a compute wave, then a workgroup per piece of the layers)
        auto chain = [&](auto kern, uint32_t cells, uint32_t threads, const uint32_t* gate) -> int {
            const uint32_t keepers = (uint32_t)(cap / cells + 1);
            const Pieces pieces(lo.L);
            const uint32_t others = pieces.fours + pieces.ones * (uint32_t)(cap / BLOCK_CELLS + 1);
            KLAUNCH(p, s, "k_dp_chain", kern, dim3(keepers + others), dim3(threads), ab, dl, rows_g, rstride, keepers, gate);
            KLAUNCH(p, s, "k_dp_walk", k_dp_walk, dim3(1), dim3(1024), ab, (const double*)(rows_g + (size_t)lo.L * rstride),
                    (const uint32_t*)dl.bad, (int32_t)KIMAD_ERR_INFEASIBLE, (int32_t)KIMAD_ERR_NONFINITE, (int32_t)KIMAD_ERR_INTERNAL, sl, gate);
            return KIMAD_OK;
        };
        auto chain_by_size = [&](const uint32_t* gate) -> int {
            if (cap + 1 <= 1024 && lo.L > CHAIN_NARROW_L) return chain(k_dp_chain<1024, 4, 2>, 64, chain_threads(4, 2), gate);
            if (cap + 1 <= 1024) return chain(k_dp_chain<1024, 8, 2>, 128, chain_threads(8, 2), gate);
            if (cap + 1 <= 2048) return chain(k_dp_chain<2048, 8, 3>, 128, chain_threads(8, 3), gate);
            return chain(k_dp_chain<DP_ROW_MAX, 4, 5>, 64, chain_threads(4, 5), gate);
        };
        if (tree) {
            TreeBuffers tb = ws.tree;
            tb.S = tree_segments(choices, cap + 1 <= 1024 ? TREE_FEW : TREE_FEW_LONG);
            if (cap + 1 <= 1024) {
                KLAUNCH(p, s, "k_dp_segments", k_dp_segments<1024>, dim3(tb.S + (lo.L + 15u) / 16u), dim3(SEGMENT_THREADS), ab, dl, tb);
            } else {
                KLAUNCH(p, s, "k_dp_segments", k_dp_segments<DP_ROW_MAX>, dim3(tb.S + (lo.L + 15u) / 16u), dim3(SEGMENT_THREADS), ab, dl, tb);
            }
            for (uint32_t first = tb.S / 2u; first >= 2u; first >>= 1) {
                auto join = [&](auto kern, uint32_t costs) -> int {
                    KLAUNCH(p, s, "k_dp_join", kern, dim3((uint32_t)(cap / costs + 1), first), dim3(JOIN_THREADS), tb, first);
                    return KIMAD_OK;
                };
                const int rc = cap + 1 <= 1024 ? join(k_dp_join<1024, 16, 4>, 16)
                             : first * (cap / 64 + 1) < JOIN_WIDE_WGS ? join(k_dp_join<DP_ROW_MAX, 32, 4>, 32) : join(k_dp_join<DP_ROW_MAX, 64, 8>, 64);
                if (rc) return rc;
            }
            if (cap + 1 <= 1024) {
                KLAUNCH(p, s, "k_dp_path", k_dp_path<true>, dim3(tb.S), dim3(PATH_THREADS), ab, dl, tb, (int32_t)KIMAD_ERR_INFEASIBLE,
                        (int32_t)KIMAD_ERR_NONFINITE, sl);
            } else {
                KLAUNCH(p, s, "k_dp_path", k_dp_path<false>, dim3(tb.S), dim3(PATH_THREADS), ab, dl, tb, (int32_t)KIMAD_ERR_INFEASIBLE,
                        (int32_t)KIMAD_ERR_NONFINITE, sl);
            }
            return chain_by_size(tb.head + 3);
        }
        KLAUNCH(p, s, "k_dp_prep", k_dp_prep, dim3(lo.L), dim3(64), ab, dl, band ? 1u : 0u, band ? (double*)nullptr : rows_g,
                (uint64_t)rstride, 0u, (double*)nullptr, (uint32_t)ROUTE_ROWS);
        if (band) {
            // the recurrence inside the band of cells that Lagrangian bounds leave (same result, a fraction of the cells)
            BandBuffers bb = ws.band;
            bb.table = rows_g;                    // (a stored row has at least BAND_NLAM cells)
            KLAUNCH(p, s, "k_dp_bounds", k_dp_bounds, dim3(1), dim3(BOUNDS_THREADS), ab, dl, bb);
            KLAUNCH(p, s, "k_dp_banded", k_dp_banded, dim3(1), dim3(BANDED_THREADS), ab, dl, bb, rows_g, rstride,
                    (int32_t)KIMAD_ERR_INFEASIBLE, (int32_t)KIMAD_ERR_NONFINITE, sl);
            return KIMAD_OK;
        }
        return chain_by_size(nullptr);
    } else if (ws.all_rows) {
        const uint64_t pitch = chain_long_pitch(cap + 1);
        const bool halves = lo.L >= (lo.J <= HALVES_FEW_J && cap + 1 < HALVES_LONG ? HALVES_MIN_L_SHORT : HALVES_MIN_L) && lo.L <= HALVES_MAX_L && cap + 1 <= HALVES_MAX_CELLS && first_ticket == 0u &&
                            !(p->cfg.flags & KIMAD_CFG_FULL_DP);
        // (a row's filling takes several workgroups: one per 32 KB)
        const dim3 fill(lo.L, (uint32_t)(pitch / 4096 + 1));
        KLAUNCH(p, s, "k_dp_prep", k_dp_prep, fill, dim3(64), ab, ws.dl, 0u, ws.rows_g, pitch, CHAIN_PAD, halves ? ws.dl.he : (double*)nullptr,
                (uint32_t)(halves ? ROUTE_HALVES : ROUTE_ROWS));
        auto chain_of = [&](auto pair, const ChainHalves& ch) -> int {
            constexpr bool PAIR = decltype(pair)::value;
            const uint32_t* wall = ws.dl.wall;
            const dim3 block(PAIR ? 64u * CHAIN_LONG_WAVES : 64u), grid((uint32_t)(cap / block.x + 1) * (ch.order ? 2u : 1u));
            if (lo.J <= 16) KLAUNCH(p, s, "k_dp_chain", (k_dp_chain_long<1, PAIR>), grid, block, ab, wall, ws.rows_g, pitch, ch);
            else if (lo.J <= 32) KLAUNCH(p, s, "k_dp_chain", (k_dp_chain_long<2, PAIR>), grid, block, ab, wall, ws.rows_g, pitch, ch);
            else KLAUNCH(p, s, "k_dp_chain", (k_dp_chain_long<4, PAIR>), grid, block, ab, wall, ws.rows_g, pitch, ch);
            return KIMAD_OK;
        };
        auto chain = [&](const ChainHalves& ch) -> int {
            return ch.order || chain_long_waves(lo.L, lo.J, cap + 1) == CHAIN_LONG_WAVES ? chain_of(std::true_type{}, ch) : chain_of(std::false_type{}, ch);
        };
        const double* last = ws.rows_g + (uint64_t)lo.L * pitch + CHAIN_PAD;
        ChainHalves ch{};
        const uint32_t* gate = nullptr;
        if (halves) {
            ch.order = at<uint32_t>(p, lo.half_order); ch.falling = ws.dl.he; ch.least[0] = ws.row0; ch.least[1] = ws.row1;
            ch.split = lo.L / 2;
            int rc = chain(ch);
            if (rc) return rc;
            double* results = ws.row0 + MEET_RESULTS;
            KLAUNCH(p, s, "k_dp_meet", k_dp_meet, dim3((uint32_t)(cap / MEET_THREADS + 1)), dim3(MEET_THREADS), ab, (const double*)ws.dl.habs,
                    (const double*)(ws.rows_g + (uint64_t)ch.split * pitch + CHAIN_PAD), last, (const double*)ws.row1, results);
            KLAUNCH(p, s, "k_dp_back", k_dp_back, dim3(2), dim3(BACK_THREADS), ab, (const double*)ws.rows_g, pitch, CHAIN_PAD, ch.split, ch.order,
                    (const uint32_t*)ws.dl.wall, ch.falling, (const uint32_t*)ws.dl.bad, (const double*)ws.row1,
                    (const double*)(results + 3 * MEET_MAX), (int32_t)KIMAD_ERR_INFEASIBLE, (int32_t)KIMAD_ERR_NONFINITE,
                    (int32_t)KIMAD_ERR_INTERNAL, sl);
            KLAUNCH(p, s, "k_dp_refill", k_dp_refill, dim3(std::min<uint32_t>(lo.L, 64u), 16), dim3(64), ab, ws.rows_g, pitch, CHAIN_PAD);
            ch.order = nullptr;
            ch.gate = gate = ws.flags + FLAG_CHAIN;
        }
        int rc = chain(ch);
        if (rc) return rc;
        KLAUNCH(p, s, "k_dp_final", k_dp_final, dim3(1), dim3(1024), ab, last, (const uint32_t*)ws.dl.bad, (int32_t)KIMAD_ERR_INFEASIBLE,
                (int32_t)KIMAD_ERR_NONFINITE, (int32_t)KIMAD_ERR_INTERNAL, sl, gate);
    } else {
        const uint32_t cell_blocks = (uint32_t)((cap + 1 + 255) / 256);
        // (clears with a kernel, not hipMemsetAsync: the call may be recorded into a graph)
        KLAUNCH(p, s, "k_zero16", k_zero16, dim3(1), dim3(256), reinterpret_cast<uint4*>(ws.flags), (uint64_t)1);
        KLAUNCH(p, s, "k_dp_init", k_dp_init, dim3(std::min<uint32_t>(cell_blocks, 1024)), dim3(256), ab);
        double* rows[2] = {ab.row0, ab.row1};
        for (uint32_t i = 0; i < lo.L; ++i) {
            KLAUNCH(p, s, "k_dp_layer", k_dp_layer, dim3(cell_blocks), dim3(256), ab, i, rows[i & 1], rows[(i + 1) & 1]);
        }
        KLAUNCH(p, s, "k_dp_final", k_dp_final, dim3(1), dim3(1024), ab, (const double*)rows[lo.L & 1], (const uint32_t*)nullptr,
                (int32_t)KIMAD_ERR_INFEASIBLE, (int32_t)KIMAD_ERR_NONFINITE, (int32_t)KIMAD_ERR_INTERNAL, sl, (const uint32_t*)nullptr);
    }
    return KIMAD_OK;
}

// The plan's compression buffers with a call's arguments.
CompressBuffers compress_buffers(kimad_plan* p, const uint64_t* K, const uint64_t* offsets, uint32_t* idx_out, void* val_out,
                                 uint64_t capacity_pairs, int32_t* status_out) {
    CompressBuffers cb = p->cb;
    cb.K = K; cb.offsets = offsets; cb.idx_out = idx_out; cb.val_out = static_cast<float*>(val_out);
    cb.value_f16 = p->cfg.value_format == KIMAD_VALUES_F16 ? 1u : 0u;
    cb.capacity_pairs = capacity_pairs; cb.status = status_out;
    return cb;
}

// The compression's kernels behind the look-up.
int enqueue_compress(kimad_plan* p, const CompressBuffers& cb, hipStream_t s) {
    const Layout& lo = p->lo;
    hipStream_t ss = s;
    const bool with_bases = lo.B && lo.S <= SMALL_BESIDE;
    if (lo.S && !with_bases) {
        ss = fork_side(p, s);                 // after the lookup: the small layers read its verdict
        KLAUNCH(p, ss, "k_small_compress", k_small_compress, dim3(lo.S), dim3(SMALL_THREADS), cb);
    }
    if (lo.B) {
        const uint32_t* chunk_big = at<uint32_t>(p, lo.chunk_big);
        const uint32_t cblocks = (lo.nchunks + CHUNKS_PER_WG - 1) / CHUNKS_PER_WG;
        const uint32_t nblocks = (lo.nchunks + 256u / SUB_COUNT - 1) / (256u / SUB_COUNT);   // where candidates are only counted
        const uint32_t hblocks = (lo.nchunks + 256u / SUB_HIST - 1) / (256u / SUB_HIST);      // and where they are histogrammed
        KLAUNCH(p, s, "k_candidates", k_candidates, dim3(hblocks + std::min<uint32_t>(lo.ntiles, 4u * FALLBACK_GRID)), dim3(256), cb,
                lo.nchunks, chunk_big, hblocks, lo.ntiles, (int32_t)KIMAD_ERR_INTERNAL);
        KLAUNCH(p, s, "k_resolve", k_resolve, dim3(lo.B), dim3(256), cb);
        // (the workgroups behind the candidates' leave after one load when no layer is served from g and h throughout)
        const uint32_t dblocks = std::min<uint32_t>(lo.ntiles, FALLBACK_GRID);
        KLAUNCH(p, s, "k_chunk_count", k_chunk_count, dim3(nblocks + dblocks), dim3(256), cb, lo.nchunks, chunk_big, nblocks, lo.ntiles);
        KLAUNCH(p, s, "k_chunk_bases", k_chunk_bases, dim3(lo.ncblk + (with_bases ? lo.S : 0u)), dim3(SMALL_THREADS), cb, lo.ncblk);
        KLAUNCH(p, s, "k_finalize", k_finalize, dim3(cblocks + dblocks), dim3(256), cb, lo.nchunks, chunk_big, cblocks, lo.ntiles);
    }
    return join_side(p, s, ss);
}

}  // namespace

extern "C" {

int kimad_workspace_bytes(const uint64_t* n, uint32_t L, uint32_t J, const kimad_config_t* cfg, uint64_t* bytes_out) {
    if (!bytes_out) return KIMAD_ERR_INVALID_ARG;
    Layout lo;
    const int rc = make_layout(n, L, J, normalise(cfg), lo, nullptr);
    if (rc) return rc;
    *bytes_out = lo.total;
    return KIMAD_OK;
}

int kimad_plan_create(const kimad_layer_t* layers, uint32_t L, const double* ratios, uint32_t J,
                      const kimad_config_t* cfg, void* workspace, uint64_t workspace_bytes, void* stream,
                      kimad_plan_t** plan_out) {
    if (!layers || !ratios || !workspace || !plan_out) return KIMAD_ERR_INVALID_ARG;
    if (L == 0 || L > 65535 || J == 0 || J > KIMAD_MAX_J) return KIMAD_ERR_INVALID_ARG;
    if (cfg && cfg->value_format > KIMAD_VALUES_F16) return KIMAD_ERR_INVALID_ARG;
    if (((uintptr_t)workspace) % ALIGN) return KIMAD_ERR_INVALID_ARG;
    for (uint32_t j = 0; j < J; ++j) {
        if (!(ratios[j] > 0.0) || !(ratios[j] <= 1.0)) return KIMAD_ERR_INVALID_ARG;
        if (j && !(ratios[j] > ratios[j - 1])) return KIMAD_ERR_INVALID_ARG;
    }
    std::vector<uint64_t> n(L);
    for (uint32_t i = 0; i < L; ++i) {
        if (!layers[i].g || !layers[i].h) return KIMAD_ERR_INVALID_ARG;
        if (((uintptr_t)layers[i].g) % 4 || ((uintptr_t)layers[i].h) % 4) return KIMAD_ERR_INVALID_ARG;
        n[i] = layers[i].n;
    }
    kimad_plan* p = new (std::nothrow) kimad_plan();
    if (!p) return KIMAD_ERR_INVALID_ARG;
    p->cfg = normalise(cfg);
    p->ratio0 = ratios[0];
    PartTables pt;
    int rc = make_layout(n.data(), L, J, p->cfg, p->lo, &p->hl, &pt);
    if (rc) { delete p; return rc; }
    if (workspace_bytes < p->lo.least) { delete p; return KIMAD_ERR_WORKSPACE_TOO_SMALL; }
    p->all_rows = workspace_bytes >= p->lo.total;
    p->ws = static_cast<char*>(workspace);
    if (hipGetDevice(&p->device) != hipSuccess) { delete p; return KIMAD_ERR_HIP; }
    (void)static_scratch_of_current_device();   // set-up: the address of this device's fixed tables is known from here on
    const Layout& lo = p->lo;

    // host tables
    std::vector<LayerDesc> ld(L);
    std::vector<uint32_t> tile_layer(lo.ntiles ? lo.ntiles : 1), chunk_big(lo.nchunks ? lo.nchunks : 1);
    std::vector<uint32_t> chunk_first(lo.nchunks ? lo.nchunks : 1);
    std::vector<uint32_t> big_layer(lo.B + 1), small_layer(lo.S ? lo.S : 1);
    std::vector<uint64_t> big_tmp0(lo.B ? lo.B : 1);
    std::vector<uint32_t> swg_layer(lo.nswg ? lo.nswg : 1), swg_first(lo.nswg ? lo.nswg : 1);
    std::vector<uint32_t> cblk_big(lo.ncblk ? lo.ncblk : 1);
    p->ktab.resize((size_t)L * J);
    p->kmax.resize(L);
    uint32_t si = 0;
    for (uint32_t i = 0; i < L; ++i) {
        HostLayer& h = p->hl[i];
        h.mis = (uint32_t)((((uintptr_t)layers[i].g) / 4) & 3u);
        h.hvec = ((((uintptr_t)layers[i].h) / 4) & 3u) == h.mis;
        LayerDesc& d = ld[i];
        d.g = layers[i].g; d.h = layers[i].h; d.n = h.n; d.mis = h.mis; d.hvec = h.hvec; d.big = h.big;
        if (h.big >= 0) {
            // Tiles and chunks are reserved for the worst misalignment; positions past the end of
            // the layer load nothing.
            for (uint32_t t = 0; t < h.ntiles; ++t) tile_layer[h.tile0 + t] = i;
            for (uint32_t c = 0; c < h.nchunks; ++c) { chunk_big[h.chunk0 + c] = (uint32_t)h.big; chunk_first[h.chunk0 + c] = h.chunk0; }
            d.tile0 = h.tile0; d.ntiles = h.ntiles; d.chunk0 = h.chunk0; d.nchunks = h.nchunks;
            d.sstride = h.sstride; d.cblk0 = h.cblk0; d.tmp0 = h.tmp0; d.tmp_cap = h.tmp_cap; d.pad = 0;
            for (uint32_t k = 0; k < h.ncblk; ++k) cblk_big[h.cblk0 + k] = (uint32_t)h.big;
            for (uint32_t w = 0; w < h.nswg; ++w) {
                swg_layer[h.swg0 + w] = i;
                swg_first[h.swg0 + w] = w * SAMPLE_GROUPS_PER_WG;
            }
            big_layer[h.big] = i;
            big_tmp0[h.big] = h.tmp0;
        } else {
            d.tile0 = d.ntiles = d.chunk0 = d.nchunks = 0;
            d.sstride = 1; d.cblk0 = 0; d.tmp0 = 0; d.tmp_cap = 0; d.pad = 0;
            small_layer[si++] = i;
        }
        for (uint32_t j = 0; j < J; ++j) p->ktab[(size_t)i * J + j] = grid_size_K(ratios[j], h.n);
        p->kmax[i] = p->ktab[(size_t)i * J + J - 1];
    }
    const std::vector<ReduceLayer> reduce = pt.reduce_layers();
    // the halves of an allocation beyond LDS: layers that reach least first, dealt out in turn
    std::vector<uint32_t> by_reach(L), half_order;
    std::iota(by_reach.begin(), by_reach.end(), 0u);
    std::stable_sort(by_reach.begin(), by_reach.end(), [&](uint32_t a, uint32_t b) { return p->kmax[a] < p->kmax[b]; });
    for (uint32_t h = 0; h < 2; ++h)
        for (uint32_t i = 1 - h; i < L; i += 2) half_order.push_back(by_reach[i]);
    hipStream_t s = static_cast<hipStream_t>(stream);
    auto up = [&](uint64_t off, const void* src, size_t bytes) {
        return hipMemcpyAsync(p->ws + off, src, bytes, hipMemcpyHostToDevice, s) == hipSuccess;
    };
    bool ok = up(lo.layers, ld.data(), sizeof(LayerDesc) * L) && up(lo.ktab, p->ktab.data(), 4ull * L * J) &&
              up(lo.tile_layer, tile_layer.data(), 4ull * tile_layer.size()) &&
              up(lo.chunk_big, chunk_big.data(), 4ull * chunk_big.size()) &&
              up(lo.chunk_first, chunk_first.data(), 4ull * chunk_first.size()) &&
              up(lo.big_layer, big_layer.data(), 4ull * big_layer.size()) &&
              up(lo.big_tmp0, big_tmp0.data(), 8ull * big_tmp0.size()) &&
              up(lo.shares, pt.shares.data(), sizeof(MainShare) * pt.shares.size()) &&
              (reduce.empty() || up(lo.reduce_layers, reduce.data(), sizeof(ReduceLayer) * reduce.size())) &&
              up(lo.small_layer, small_layer.data(), 4ull * small_layer.size()) &&
              up(lo.swg_layer, swg_layer.data(), 4ull * swg_layer.size()) &&
              up(lo.swg_first, swg_first.data(), 4ull * swg_first.size()) &&
              up(lo.cblk_big, cblk_big.data(), 4ull * cblk_big.size()) &&
              up(lo.half_order, half_order.data(), 4ull * L);
    ok = ok && hipStreamSynchronize(s) == hipSuccess;     // host vectors go out of scope below
    if (!ok) { delete p; return KIMAD_ERR_HIP; }

    ProfileBuffers& pb = p->pb;
    pb.layers = at<LayerDesc>(p, lo.layers);
    pb.tile_layer = at<uint32_t>(p, lo.tile_layer);
    pb.big_layer = at<uint32_t>(p, lo.big_layer);
    pb.small_layer = at<uint32_t>(p, lo.small_layer);
    pb.tile_elems = lo.tile_elems;
    pb.cnt1 = at<uint32_t>(p, lo.cnt1); pb.sq1 = at<uint64_t>(p, lo.sq1);
    pb.lut1 = at<uint8_t>(p, lo.lut1); pb.nslots = at<uint32_t>(p, lo.nslots); pb.slot_bin = at<uint32_t>(p, lo.slot_bin);
    pb.slot_cnt = at<uint32_t>(p, lo.slot_cnt); pb.slot_sq = at<uint64_t>(p, lo.slot_sq);
    pb.cnt2 = at<uint32_t>(p, lo.cnt2); pb.sq2 = at<uint64_t>(p, lo.sq2);
    pb.tgt_slot = at<uint32_t>(p, lo.tgt_slot); pb.tgt_r = at<uint32_t>(p, lo.tgt_r);
    pb.tgt_above1 = at<uint32_t>(p, lo.tgt_above1); pb.tgt_below = at<double>(p, lo.tgt_below);
    pb.sel_prefix = at<uint32_t>(p, lo.sel_prefix); pb.sel_above = at<uint32_t>(p, lo.sel_above);
    pb.sel_amb = at<uint32_t>(p, lo.sel_amb); pb.diag = at<uint32_t>(p, lo.diag);
    pb.fresh = at<uint32_t>(p, lo.fresh);
    pb.hprev = at<uint32_t>(p, lo.hprev); pb.gprev = at<unsigned long long>(p, lo.gprev);
    pb.layer_flag = at<uint32_t>(p, lo.layer_flag);
    pb.tiles_done = at<uint32_t>(p, lo.tiles_done);
    pb.pool_prefix = at<uint32_t>(p, lo.pool_prefix); pb.pool_big = at<uint32_t>(p, lo.pool_big);
    pb.pool_t0 = at<uint32_t>(p, lo.pool_t0); pb.pool_cnt = at<uint32_t>(p, lo.pool_cnt);
    pb.pool_hist = at<uint32_t>(p, lo.pool_hist); pb.pool_cap = lo.pool_cap;
    pb.tgt_unsel = at<uint32_t>(p, lo.tgt_unsel); pb.tgt_base = at<double>(p, lo.tgt_base);
    pb.state = at<LayerState>(p, lo.state); pb.big_tmp0 = at<uint64_t>(p, lo.big_tmp0);
    pb.parts = at<unsigned long long>(p, lo.parts); pb.part_head = at<uint32_t>(p, lo.part_head); pb.shares = at<MainShare>(p, lo.shares);
    pb.reduce_layers = at<ReduceLayer>(p, lo.reduce_layers);
    pb.chunk_big = at<uint32_t>(p, lo.chunk_big); pb.chunk_first = at<uint32_t>(p, lo.chunk_first); pb.nchunks_total = lo.nchunks;
    pb.swg_layer = at<uint32_t>(p, lo.swg_layer); pb.swg_first = at<uint32_t>(p, lo.swg_first);
    pb.shist = at<uint32_t>(p, lo.shist); pb.ghist = at<unsigned long long>(p, lo.ghist);
    pb.lutc = at<uint8_t>(p, lo.lutc); pb.cursor = at<uint32_t>(p, lo.cursor);
    pb.spill_over = at<uint32_t>(p, lo.spill_over);
    pb.rec_start = at<uint32_t>(p, lo.rec_start); pb.rec_cnt = at<uint32_t>(p, lo.rec_cnt);
    pb.tmp_x = at<float>(p, lo.tmp_x); pb.tmp_i = at<uint16_t>(p, lo.tmp_i);
    p->main_wgs = lo.main_wgs;
    // Layer states start as "nothing spilled, nothing cached".
    if (hipMemsetAsync(p->ws + lo.state, 0, sizeof(LayerState) * (uint64_t)(lo.B ? lo.B : 1), s) != hipSuccess ||
        hipMemsetAsync(p->ws + lo.zero2_begin, 0, lo.zero2_end - lo.zero2_begin, s) != hipSuccess ||
        hipMemsetAsync(p->ws + lo.band_info, 0, 4 * INFO_WORDS, s) != hipSuccess ||
        hipMemsetAsync(p->ws + lo.fresh, 0, 16, s) != hipSuccess ||
        hipMemsetAsync(p->ws + lo.gprev, 0, 8ull * D1_BINS, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) { delete p; return KIMAD_ERR_HIP; }

    CompressBuffers& cb = p->cb;
    cb.layers = pb.layers; cb.chunk_layer = pb.tile_layer; cb.big_layer = pb.big_layer; cb.small_layer = pb.small_layer;
    cb.tile_elems = lo.tile_elems; cb.L = L; cb.B = lo.B; cb.J = J;
    cb.Ktab = at<uint32_t>(p, lo.ktab);
    cb.sel_prefix = pb.sel_prefix; cb.sel_above = pb.sel_above; cb.sel_amb = pb.sel_amb;
    cb.sel = at<SelRec>(p, lo.sel); cb.cursor = pb.cursor; cb.hist3 = at<uint32_t>(p, lo.hist3);
    cb.tau = at<uint32_t>(p, lo.tau); cb.quota = at<uint32_t>(p, lo.quota);
    cb.rec_start = at<uint32_t>(p, lo.rec_start); cb.rec_cnt = at<uint32_t>(p, lo.rec_cnt);
    cb.chunk_first = at<uint32_t>(p, lo.chunk_first); cb.tmp_total = lo.tmp_cap;
    cb.rec_amb = at<uint32_t>(p, lo.rec_amb); cb.c_gt = at<uint32_t>(p, lo.c_gt); cb.c_eq = at<uint32_t>(p, lo.c_eq);
    cb.o_base = at<uint32_t>(p, lo.o_base); cb.o_allow = at<uint32_t>(p, lo.o_allow);
    cb.cblk_big = at<uint32_t>(p, lo.cblk_big);
    cb.tmp_x = at<float>(p, lo.tmp_x); cb.tmp_i = at<uint16_t>(p, lo.tmp_i);
    cb.ncompact = at<uint32_t>(p, lo.ncompact);
    cb.fresh = pb.fresh;
    cb.state = pb.state;
    cb.K = nullptr; cb.offsets = nullptr; cb.idx_out = nullptr; cb.val_out = nullptr; cb.capacity_pairs = 0;
    cb.value_f16 = 0;
    cb.status = nullptr;
    if (lo.S && lo.B) {
        // default priority; without the side stream everything simply runs in order on the caller's stream
        if (hipStreamCreateWithFlags(&p->side, hipStreamNonBlocking) != hipSuccess) p->side = nullptr;
        if (p->side && (hipEventCreateWithFlags(&p->ev_fork, hipEventDisableTiming) != hipSuccess ||
                        hipEventCreateWithFlags(&p->ev_join, hipEventDisableTiming) != hipSuccess)) {
            (void)hipStreamDestroy(p->side);
            p->side = nullptr;
        }
    }
    *plan_out = p;
    return KIMAD_OK;
}

int kimad_plan_destroy(kimad_plan_t* plan) {
    delete plan;
    return KIMAD_OK;
}

int kimad_plan_grid_sizes(const kimad_plan_t* plan, uint64_t* K_table_out) {
    if (!plan || !K_table_out) return KIMAD_ERR_INVALID_ARG;
    for (size_t t = 0; t < plan->ktab.size(); ++t) K_table_out[t] = plan->ktab[t];
    return KIMAD_OK;
}

int kimad_profile(kimad_plan_t* p, double* err_table, uint64_t budget_hint_bytes, void* stream) {
    if (!p || !err_table) return KIMAD_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const Layout& lo = p->lo;
    mark(p, s, "begin");
    hipStream_t ss = s;
    int rc;
    if (p->cfg.flags & KIMAD_CFG_CLASSIC_PROFILE) {
        // (the clearing comes before the fork: the small layers' kernel on the side stream marks the profile as
        // fresh, and in a plan without tiled layers nothing marks it again)
        rc = zero_range(p, lo.zero1_begin, lo.zero1_end, s);
        if (!rc) rc = launch_small_profile(p, err_table, s, &ss);
        if (!rc) rc = run_select_passes(p, at<uint32_t>(p, lo.ktab), lo.J, err_table, s, 1u, false);
    } else {
        rc = run_single_pass(p, at<uint32_t>(p, lo.ktab), lo.J, err_table, budget_hint_bytes / p->cfg.pair_bytes, s, &ss);
    }
    const int rj = join_side(p, s, ss);       // always join, also after an error
    return rc ? rc : rj;
}

int kimad_allocate(kimad_plan_t* p, const double* err_table, uint64_t budget_bytes, int32_t* j_out, uint64_t* K_out,
                   uint64_t* offsets_out, int32_t* status_out, void* stream) {
    if (!p || !err_table || !j_out || !K_out || !offsets_out || !status_out) return KIMAD_ERR_INVALID_ARG;
    const AllocScratch ws = plan_scratch(p);
    return enqueue_allocate(p, ws, err_table, budget_bytes, j_out, K_out, offsets_out, status_out,
                            static_cast<hipStream_t>(stream));
}

int kimad_allocate_static(kimad_plan_t* p, const double* err_table, uint64_t budget_bytes, int32_t* j_out,
                          uint64_t* K_out, uint64_t* offsets_out, int32_t* status_out, void* stream) {
    if (!p || !err_table || !j_out || !K_out || !offsets_out || !status_out) return KIMAD_ERR_INVALID_ARG;
    const Layout& lo = p->lo;
    if (lo.L > KIMAD_STATIC_MAX_L) return KIMAD_ERR_STATIC_LIMIT;
    unsigned char* base = static_scratch_of_current_device();
    if (!base) return KIMAD_ERR_HIP;
    // Fixed carving of the array for the largest case it admits (KIMAD_STATIC_MAX_L layers, KIMAD_MAX_J
    // ratios, rows of KIMAD_STATIC_MAX_CELLS cost cells), so the offsets do not depend on the plan.
    constexpr uint64_t LJ = (uint64_t)KIMAD_STATIC_MAX_L * KIMAD_MAX_J;
    constexpr uint64_t CELLS = KIMAD_STATIC_MAX_CELLS;
    uint64_t off = 0;
    auto take = [&](uint64_t bytes) { unsigned char* q = base + off; off = align_up(off + bytes); return q; };
    AllocScratch ws;
    ws.row0 = nullptr; ws.row1 = nullptr;                       // only the per-layer-launch path uses them
    ws.choice = reinterpret_cast<uint8_t*>(take((uint64_t)KIMAD_STATIC_MAX_L * CELLS));
    ws.cprev = reinterpret_cast<uint16_t*>(take(2ull * Pieces(KIMAD_STATIC_MAX_L).count() * CELLS));
    ws.flags = reinterpret_cast<uint32_t*>(take(4 * DP_FLAGS));
    ws.dl.wall = reinterpret_cast<uint32_t*>(take(4 * LJ)); ws.dl.w = reinterpret_cast<uint32_t*>(take(4 * LJ));
    ws.dl.jj = reinterpret_cast<uint32_t*>(take(4 * LJ)); ws.dl.e = reinterpret_cast<double*>(take(16 * LJ));
    ws.dl.n = reinterpret_cast<uint32_t*>(take(4ull * KIMAD_STATIC_MAX_L));
    ws.dl.bad = reinterpret_cast<uint32_t*>(take(4ull * KIMAD_STATIC_MAX_L));
    ws.dense_E = reinterpret_cast<double*>(take(8 * LJ)); ws.dense_Kcost = reinterpret_cast<uint32_t*>(take(4 * LJ));
    ws.dense_Kout = reinterpret_cast<uint32_t*>(take(4 * LJ));
    ws.band.lo = reinterpret_cast<uint32_t*>(take(4ull * (KIMAD_STATIC_MAX_L + 1)));
    ws.band.hi = reinterpret_cast<uint32_t*>(take(4ull * (KIMAD_STATIC_MAX_L + 1)));
    ws.band.info = reinterpret_cast<uint32_t*>(take(4 * INFO_WORDS));
    ws.band.live = reinterpret_cast<uint32_t*>(take(4ull * KIMAD_STATIC_MAX_L));
    ws.dl.he = reinterpret_cast<double*>(take(8 * LJ)); ws.dl.hw = reinterpret_cast<uint32_t*>(take(4 * LJ));
    ws.dl.hn = reinterpret_cast<uint32_t*>(take(4ull * KIMAD_STATIC_MAX_L));
    ws.dl.habs = reinterpret_cast<double*>(take(8ull * KIMAD_STATIC_MAX_L));
    ws.rows_g = reinterpret_cast<double*>(take(8ull * (KIMAD_STATIC_MAX_L + 1) * CELLS));
    ws.rstride = (uint32_t)CELLS;
    ws.max_cells = CELLS;
    ws.all_rows = false;                                        // (rows of this length fit LDS)
    ws.tree = TreeBuffers{};
    static_assert(KIMAD_STATIC_MAX_CELLS == 1024, "a stored row holds the cells of k_dp_chain's whole workgroups");
    if (off > STATIC_SCRATCH_BYTES) return KIMAD_ERR_INTERNAL;
    const int rc = enqueue_allocate(p, ws, err_table, budget_bytes, j_out, K_out, offsets_out, status_out,
                                    static_cast<hipStream_t>(stream));
    return rc == KIMAD_ERR_INVALID_ARG ? KIMAD_ERR_STATIC_LIMIT : rc;   // the one argument left to reject: rows too long
}

int kimad_compress_ef(kimad_plan_t* p, const uint64_t* K, const uint64_t* offsets, uint32_t* idx_out, void* val_out,
                      uint64_t capacity_pairs, uint32_t flags, int32_t* status_out, void* stream) {
    if (!p || !K || !offsets || !idx_out || !val_out || !status_out) return KIMAD_ERR_INVALID_ARG;
    if (flags & ~KIMAD_REUSE_PROFILE) return KIMAD_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const Layout& lo = p->lo;
    CompressBuffers cb = compress_buffers(p, K, offsets, idx_out, val_out, capacity_pairs, status_out);
    mark(p, s, "begin");
    const bool reuse = (flags & KIMAD_REUSE_PROFILE) != 0;
    const bool single = !(p->cfg.flags & KIMAD_CFG_CLASSIC_PROFILE) && lo.nchunks >= SINGLE_SELECT_CHUNKS &&
                        lo.nchunks >= SINGLE_SELECT_PER_LAYER * lo.B;
    if (!reuse) {
        // Select from scratch, one target per layer: by the single pass over g and h that the profile takes, whose
        // candidates then serve the selection, or by two histogram passes and a compaction (SINGLE_SELECT_CHUNKS).
        uint32_t* ksel = at<uint32_t>(p, lo.ksel);
        KLAUNCH(p, s, "k_make_ksel", k_make_ksel, dim3((lo.L + 255) / 256), dim3(256), K, cb.layers, lo.L, ksel);
        hipStream_t unused = s;
        const int rc = single ? run_single_pass(p, ksel, 1, nullptr, 0, s, &unused) : run_select_passes(p, ksel, 1, nullptr, s);
        if (rc) return rc;
        cb.Ktab = ksel;
        cb.J = 1;
    }
    // (the last-digit histograms are zero here: k_resolve clears what it has read)
    KLAUNCH(p, s, "k_lookup", k_lookup, dim3(1), dim3(256), cb, (int32_t)KIMAD_ERR_OFFGRID,
            (int32_t)KIMAD_ERR_BAD_OFFSETS, (int32_t)KIMAD_ERR_STALE_PROFILE,
            (uint32_t)(reuse ? 1u : 0u), (uint32_t)(reuse || single ? 1u : 0u));
    return enqueue_compress(p, cb, s);
}

int kimad_step(kimad_plan_t* p, uint64_t budget_bytes, double* err_table, int32_t* j_out, uint64_t* K_out,
               uint64_t* offsets_out, uint32_t* idx_out, void* val_out, uint64_t capacity_pairs, int32_t* status_out,
               void* stream) {
    if (!status_out) return KIMAD_ERR_INVALID_ARG;
    int rc = kimad_profile(p, err_table, budget_bytes, stream);
    if (rc) return rc;
    if (!idx_out || !val_out) {
        // (the allocation is there, and the compression refuses)
        rc = kimad_allocate(p, err_table, budget_bytes, j_out, K_out, offsets_out, status_out, stream);
        return rc ? rc : KIMAD_ERR_INVALID_ARG;
    }
    if (!j_out || !K_out || !offsets_out) return KIMAD_ERR_INVALID_ARG;
    // On an allocation failure K and offsets are zero-filled, so the compression writes nothing.
    hipStream_t s = static_cast<hipStream_t>(stream);
    StepLookup sl{};
    sl.cb = compress_buffers(p, K_out, offsets_out, idx_out, val_out, capacity_pairs, status_out + 1);
    sl.j = j_out;
    sl.err_offgrid = KIMAD_ERR_OFFGRID; sl.err_offsets = KIMAD_ERR_BAD_OFFSETS; sl.err_stale = KIMAD_ERR_STALE_PROFILE; sl.on = 1u;
    rc = enqueue_allocate(p, plan_scratch(p), err_table, budget_bytes, j_out, K_out, offsets_out, status_out, s, CHAIN_POLLS, 0u, sl);
    return rc ? rc : enqueue_compress(p, sl.cb, s);
}

int kimad_profile_diagnostics(kimad_plan_t* p, uint32_t* out4, void* stream) {
    if (!p || !out4) return KIMAD_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (hipMemcpyAsync(out4, p->ws + p->lo.diag, 16, hipMemcpyDeviceToHost, s) != hipSuccess) return KIMAD_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return KIMAD_ERR_HIP;
    return KIMAD_OK;
}

int kimad_allocate_diagnostics(kimad_plan_t* p, uint32_t* out4, void* stream) {
    if (!p || !out4) return KIMAD_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (hipMemcpyAsync(out4, p->ws + p->lo.band_info, 16, hipMemcpyDeviceToHost, s) != hipSuccess) return KIMAD_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return KIMAD_ERR_HIP;
    return KIMAD_OK;
}

int kimad_allocate_route(kimad_plan_t* p, uint32_t* out2, void* stream) {
    static_assert(KIMAD_ROUTE_ROWS == ROUTE_ROWS && KIMAD_ROUTE_BAND == ROUTE_BAND && KIMAD_ROUTE_TREE == ROUTE_TREE &&
                  KIMAD_ROUTE_HALVES == ROUTE_HALVES && KIMAD_HOW_ROWS == HOW_ROWS && KIMAD_HOW_FROM_LEFT == HOW_FROM_LEFT &&
                  KIMAD_HOW_AT_ONCE == HOW_AT_ONCE, "header and kernel constants");
    if (!p || !out2) return KIMAD_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (hipMemcpyAsync(out2, at<uint32_t>(p, p->lo.band_info) + INFO_ROUTE, 8, hipMemcpyDeviceToHost, s) != hipSuccess) return KIMAD_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return KIMAD_ERR_HIP;
    return KIMAD_OK;
}

int kimad_plan_set_timing(kimad_plan_t* p, int enable) {
    if (!p) return KIMAD_ERR_INVALID_ARG;
    if (enable && p->ev.empty()) {
        p->ev.resize(MAX_EVENTS);
        p->ev_name.assign(MAX_EVENTS, "");
        for (uint32_t k = 0; k < MAX_EVENTS; ++k)
            if (hipEventCreate(&p->ev[k]) != hipSuccess) { p->ev.resize(k); p->timing = false; return KIMAD_ERR_HIP; }
    }
    p->timing = enable != 0;
    p->ev_n = 0;
    return KIMAD_OK;
}

int kimad_plan_get_timings(kimad_plan_t* p, char* names, uint32_t names_bytes, float* ms, uint32_t max_entries,
                           uint32_t* count_out) {
    if (!p || !names || !ms || !count_out) return KIMAD_ERR_INVALID_ARG;
    uint32_t n = 0;
    size_t pos = 0;
    if (p->ev_n) {
        if (hipEventSynchronize(p->ev[p->ev_n - 1]) != hipSuccess) return KIMAD_ERR_HIP;
        for (uint32_t k = 1; k < p->ev_n && n < max_entries; ++k) {
            if (std::strcmp(p->ev_name[k], "begin") == 0) continue;   // gap between two calls
            float t = 0.f;
            if (hipEventElapsedTime(&t, p->ev[k - 1], p->ev[k]) != hipSuccess) return KIMAD_ERR_HIP;
            const size_t len = std::strlen(p->ev_name[k]);
            if (pos + len + 2 > names_bytes) break;
            std::memcpy(names + pos, p->ev_name[k], len);
            pos += len;
            names[pos++] = '\n';
            ms[n++] = t;
        }
    }
    if (names_bytes) names[pos < names_bytes ? pos : names_bytes - 1] = 0;
    *count_out = n;
    p->ev_n = 0;
    return KIMAD_OK;
}

int kimad_plan_layer_states(kimad_plan_t* p, uint32_t* out, uint32_t max_layers, uint32_t* count_out, void* stream) {
    if (!p || !out || !count_out) return KIMAD_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint32_t B = std::min<uint32_t>(p->lo.B, max_layers);
    std::vector<LayerState> st(B ? B : 1);
    std::vector<SelRec> sel(B ? B : 1);
    if (B) {
        if (hipMemcpyAsync(st.data(), p->ws + p->lo.state, sizeof(LayerState) * B, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipMemcpyAsync(sel.data(), p->ws + p->lo.sel, sizeof(SelRec) * B, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess) return KIMAD_ERR_HIP;
    }
    uint32_t b = 0;
    for (uint32_t i = 0; i < p->lo.L && b < B; ++i) {
        if (p->hl[i].big < 0) continue;
        uint32_t* o = out + 8 * (size_t)b;
        o[0] = i; o[1] = st[b].spill_bin; o[2] = st[b].nslots_d; o[3] = st[b].nslots_t;
        o[4] = st[b].redo; o[5] = st[b].spill_cnt; o[6] = st[b].spill_valid; o[7] = sel[b].mode;
        ++b;
    }
    *count_out = b;
    return KIMAD_OK;
}

int kimad_server_apply(const kimad_payload_t* payloads, float* const* u_hat, const double* weights, uint32_t M,
                       const uint64_t* layer_start, uint32_t L, uint64_t d, float* x, double gamma,
                       int32_t* status_out, void* stream) {
    static_assert(KIMAD_MAX_WORKERS == MAX_WORKERS, "header and kernel constants");
    if (!payloads || !u_hat || !weights || !layer_start || M == 0 || M > KIMAD_MAX_WORKERS || L == 0 || d == 0 ||
        !status_out)
        return KIMAD_ERR_INVALID_ARG;
    ServerArgs a{};
    DecodeArgs da{};
    bool vec_ok = x && (reinterpret_cast<uintptr_t>(x) % 16 == 0);
    bool apart = true;                           // no two workers' estimators share memory
    uint64_t pairs = 0;                          // largest payload capacity
    for (uint32_t m = 0; m < M; ++m) {
        if (!payloads[m].idx || !payloads[m].val || !payloads[m].offsets || !u_hat[m]) return KIMAD_ERR_INVALID_ARG;
        if (payloads[m].value_format > KIMAD_VALUES_F16) return KIMAD_ERR_INVALID_ARG;
        a.u_hat[m] = u_hat[m]; a.w[m] = weights[m];
        da.idx[m] = payloads[m].idx; da.val[m] = static_cast<const float*>(payloads[m].val); da.off[m] = payloads[m].offsets;
        da.capacity_pairs[m] = payloads[m].capacity_pairs; da.u_hat[m] = u_hat[m];
        if (payloads[m].value_format == KIMAD_VALUES_F16) da.f16 |= 1u << m;
        vec_ok = vec_ok && (reinterpret_cast<uintptr_t>(u_hat[m]) % 16 == 0);
        pairs = std::max<uint64_t>(pairs, payloads[m].capacity_pairs);
        for (uint32_t k = 0; k < m; ++k) {
            const uintptr_t p0 = reinterpret_cast<uintptr_t>(u_hat[m]), p1 = reinterpret_cast<uintptr_t>(u_hat[k]);
            if ((p0 > p1 ? p0 - p1 : p1 - p0) / 4 < d) apart = false;
        }
    }
    a.M = M; a.d = d;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, s, status_out, M, 0);
    if (hipGetLastError() != hipSuccess) return KIMAD_ERR_HIP;
    // payload sizes live on the device: a grid for the capacity, of at most 1024 workgroups a worker, strides over
    // whatever the worker sent.  Workers whose estimators share memory are decoded one after another.
    const uint32_t dblocks = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((pairs + 255) / 256, 1024));
    for (uint32_t m = 0; m < M; m += apart ? M : 1u) {
        hipLaunchKernelGGL(k_server_decode, dim3(dblocks, apart ? M : 1u), dim3(256), 0, s, da, m, layer_start, L, d, status_out,
                           (int32_t)KIMAD_ERR_BAD_PAYLOAD);
        if (hipGetLastError() != hipSuccess) return KIMAD_ERR_HIP;
    }
    if (x) {
        const uint64_t work = (d + 3) / 4;
        // one quad per thread: measured 15 % faster here than a grid-stride loop over fewer blocks
        const uint32_t blocks = (uint32_t)std::min<uint64_t>((work + 255) / 256, 1ull << 22);
        if (model_stores_stream(M, d))
            hipLaunchKernelGGL(k_server_step<true>, dim3(blocks), dim3(256), 0, s, a, x, gamma, vec_ok ? 1u : 0u);
        else
            hipLaunchKernelGGL(k_server_step<false>, dim3(blocks), dim3(256), 0, s, a, x, gamma, vec_ok ? 1u : 0u);
        if (hipGetLastError() != hipSuccess) return KIMAD_ERR_HIP;
    }
    return KIMAD_OK;
}

int kimad_error_at(kimad_plan_t* p, const uint64_t* K, double* err_out, void* stream) {
    if (!p || !K || !err_out) return KIMAD_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const Layout& lo = p->lo;
    mark(p, s, "begin");
    uint32_t* ksel = at<uint32_t>(p, lo.ksel);
    KLAUNCH(p, s, "k_make_ksel", k_make_ksel, dim3((lo.L + 255) / 256), dim3(256), K, (const LayerDesc*)p->pb.layers, lo.L, ksel);
    hipStream_t ss = s;
    int rc = launch_small_profile(p, err_out, s, &ss, ksel, 1u);
    if (!rc) rc = run_select_passes(p, ksel, 1, err_out, s, 0u);   // overwrites the grid profile's cache (k_lookup sees it as gone)
    const int rj = join_side(p, s, ss);
    return rc ? rc : rj;
}

int kimad_uniform_sizes(const uint64_t* n, uint32_t L, uint64_t budget_bytes, uint32_t pair_bytes, uint64_t* K_out,
                        uint64_t* pairs_out) {
    if (!n || !K_out || L == 0) return KIMAD_ERR_INVALID_ARG;
    if (pair_bytes == 0) pair_bytes = 8;
    uint64_t d = 0;
    for (uint32_t i = 0; i < L; ++i) {
        if (n[i] == 0 || n[i] > KIMAD_MAX_N) return KIMAD_ERR_INVALID_ARG;
        d += n[i];
    }
    const uint64_t P = budget_bytes / pair_bytes;
    const double rho = std::min(1.0, (double)P / (double)d);
    for (uint32_t i = 0; i < L; ++i) K_out[i] = rho > 0.0 ? grid_size_K(rho, n[i]) : 0;
    if (pairs_out) *pairs_out = std::min(P, d);
    return KIMAD_OK;
}

int kimad_payload_layer_counts(const uint32_t* idx, uint64_t pairs, const uint64_t* layer_start, uint32_t L,
                               uint64_t* counts_out, void* stream) {
    if (!idx || !layer_start || !counts_out || L == 0) return KIMAD_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(k_layer_counts, dim3((L + 255) / 256), dim3(256), 0, s, idx, pairs, layer_start, L, counts_out);
    return hipGetLastError() == hipSuccess ? KIMAD_OK : KIMAD_ERR_HIP;
}

int kimad_selftest_wave_primitives(const uint32_t* in_u32, const double* in_f64, uint32_t* out_u32, double* out_f64,
                                   void* stream) {
    if (!in_u32 || !in_f64 || !out_u32 || !out_f64) return KIMAD_ERR_INVALID_ARG;
    hipLaunchKernelGGL(k_selftest_wave, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream), in_u32, in_f64, out_u32,
                       out_f64);
    return hipGetLastError() == hipSuccess ? KIMAD_OK : KIMAD_ERR_HIP;
}

int kimad_selftest_allocate_withheld(kimad_plan_t* p, const double* err_table, uint64_t budget_bytes, int32_t* j_out,
                                     uint64_t* K_out, uint64_t* offsets_out, int32_t* status_out, uint32_t polls,
                                     uint32_t* given_up_out, void* stream) {
    if (!p || !err_table || !j_out || !K_out || !offsets_out || !status_out || !given_up_out || polls == 0) return KIMAD_ERR_INVALID_ARG;
    const AllocScratch ws = plan_scratch(p);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int rc = enqueue_allocate(p, ws, err_table, budget_bytes, j_out, K_out, offsets_out, status_out, s, std::min(polls, CHAIN_POLLS), 1u);
    if (rc) return rc;
    return hipMemcpyAsync(given_up_out, ws.flags + 2, 4, hipMemcpyDeviceToDevice, s) == hipSuccess ? KIMAD_OK : KIMAD_ERR_HIP;
}

uint64_t kimad_budget_bytes(double bandwidth_bits_per_s, double t_seconds, double t_comp_seconds, double alpha,
                            uint64_t cap_bytes) {
    const double B = bandwidth_bits_per_s, t = t_seconds, tc = t_comp_seconds;
    if (!(B > 0.0) || !(t > tc) || !(alpha >= 0.0) || std::isinf(B) || std::isinf(t)) return 0;
    const double c_bits = B * (t - tc) / (1.0 + alpha);
    const double bytes = std::floor(c_bits / 8.0);
    uint64_t out = bytes >= 18446744073709551615.0 ? ~0ull : (uint64_t)bytes;
    if (cap_bytes && out > cap_bytes) out = cap_bytes;
    return out;
}

const char* kimad_strerror(int status) {
    switch (status) {
        case KIMAD_OK: return "ok";
        case KIMAD_ERR_INVALID_ARG: return "invalid argument";
        case KIMAD_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
        case KIMAD_ERR_HIP: return "HIP runtime error";
        case KIMAD_ERR_INFEASIBLE: return "budget below the cheapest allocation";
        case KIMAD_ERR_NONFINITE: return "error table holds a non-finite entry";
        case KIMAD_ERR_OFFGRID: return "K is not one of the layer's grid sizes";
        case KIMAD_ERR_INTERNAL: return "internal error: candidate region overflow, or the allocation gave a wait up";
        case KIMAD_ERR_BAD_OFFSETS: return "K/offsets do not fit the payload capacity";
        case KIMAD_ERR_STALE_PROFILE: return "KIMAD_REUSE_PROFILE without a profile of the current g - h";
        case KIMAD_ERR_BAD_PAYLOAD: return "payload offsets or indices do not fit the layers";
        case KIMAD_ERR_TABLES_TOO_LARGE: return "exact cost axis without a budget limit: the allocation's tables would exceed 4 GiB";
        case KIMAD_ERR_STATIC_LIMIT: return "too many layers or cost cells for the fixed tables of kimad_allocate_static";
        default: return "unknown status";
    }
}

const char* kimad_version(void) { return "kimad-gfx950 0.1"; }

}  // extern "C"
