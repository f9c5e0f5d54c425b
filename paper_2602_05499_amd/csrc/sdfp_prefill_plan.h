// The cut of a prompt into panels, the tiles of its GEMMs and the counts of their pipeline, and which kernel runs a panel's
// attention (host arithmetic only).
#pragma once
#include <algorithm>
#include <cstddef>

namespace sdfp {

// One panel: M rows from absolute position pos0, Hkv KV heads of head_dim hd (64 or 128) with grp query heads each.
struct PfAttnPanel {
    int hd, Hkv, grp, M, pos0;
    int n_cu;          // compute units
    int wg_valu;       // workgroups k_pf_attn may use (regions of split partials)
    int wg_mx;         // workgroups k_pf_attn_mx may use (slots of split partials)
};
constexpr int PF_CHUNK = 16, PF_SPLIT = 128, PF_MX_TILES = 4;   // rows of a chunk, positions of a split, tiles of a k_pf_attn_mx workgroup

// Queries of a k_pf_attn_mx workgroup whose statistics, 8 bytes per split, its LDS holds at a time during the merge; 0: not one.
constexpr int pf_mx_queries_in_lds(int lds_bytes, int n_splits) {
    const int fit = lds_bytes / 8 / n_splits, all = PF_MX_TILES * PF_CHUNK;
    return fit < all ? fit : all;
}

inline int pf_chunk_rows(const PfAttnPanel& p, int c) { return std::min(PF_CHUNK, p.M - c * PF_CHUNK); }
inline int pf_chunk_splits(const PfAttnPanel& p, int c) {
    return (p.pos0 + c * PF_CHUNK + pf_chunk_rows(p, c) + PF_SPLIT - 1) / PF_SPLIT;
}

// Both kernels are chains of latencies: a workgroup's time hardly depends on how many others run, and a launch takes as long
// as its longest workgroup, or the longest sequence of them where they do not all fit at once.  Times in us, fitted to both
// kernels' times over 1..40 KV heads x 1..8 query heads, 5 to 1568 rows (within 10 % of most; it is the comparison that
// counts).  Both sides measured, head_dim 128:
//   4 x 1 heads:  128 rows 24 / 32 (valu / mx), 256 rows 38 / 41, 512 rows 67 / 68, the 512 rows behind 512 124 / 121, one row
//                 behind 512 23 / 71, 16 rows behind 512 76 / 79, 16 behind 1024 135 / 130
//   32 x 1 heads: 129 rows 26 / 32, 256 rows 43 / 42, 288 rows 74 / 56, 512 rows 121 / 69
//   8 x 4 heads:  5 rows 31 / 28, 16 rows 87 / 31, 512 rows 241 / 69, one row behind 512 33 / 76, 8 rows behind 512 148 / 80
// head_dim 64, 4 x 1 heads: 16 rows 17 / 17, 128 rows 18 / 19, 256 rows 30 / 24, one row behind 1024 31 / 73.
//
// k_pf_attn: a workgroup per (16-row chunk, KV head), the chunk's splits one after another, queries in passes of 8; two
// workgroups share a compute unit (15 % longer).
inline double pf_valu_item_us(const PfAttnPanel& p, int c) {
    const int q = pf_chunk_rows(p, c) * p.grp, passes = (q + 7) / 8, n = pf_chunk_splits(p, c);
    return p.hd == 64 ? 4.0 + 0.19 * q + n * (1.8 + 0.8 * passes + 0.48 * q) : 4.0 + 0.35 * q + n * (2.9 + 0.7 * passes + 0.6 * q);
}
inline double pf_valu_us(const PfAttnPanel& p) {
    const int items = (p.M + PF_CHUNK - 1) / PF_CHUNK * p.Hkv, n_wg = std::min(p.wg_valu, items);
    double worst = 0.0;
    // items run in ascending chunk order, a workgroup takes every n_wg-th: the one with the last chunk, and the one with the
    // chunk before it (the last may have a row or two)
    for (int first : {items - 1, items - 1 - p.Hkv}) {
        double t = 0.0;
        for (int it = first; it >= 0; it -= n_wg) t += pf_valu_item_us(p, it / p.Hkv);
        worst = std::max(worst, t);
    }
    return worst * (n_wg > p.n_cu ? 1.15 : 1.0);
}
// k_pf_attn_mx: a workgroup per 4 tiles of a KV head, whose time is that of its longest row, however many query heads the
// rows have; one workgroup per compute unit, longest first.
inline double pf_mx_item_us(const PfAttnPanel& p, int tg, int n_tiles) {
    const int c0 = tg * PF_MX_TILES / p.grp, c1 = (std::min(n_tiles, (tg + 1) * PF_MX_TILES) - 1) / p.grp;
    const int n = pf_chunk_splits(p, c1), rows = (c1 - c0) * PF_CHUNK + pf_chunk_rows(p, c1);
    const double fill = std::min(p.grp * rows, 64) / 64.0;   // waves without rows leave more of the unit to the others
    return p.hd == 64 ? 8.2 + 7.3 * n + 3.0 * fill : 11.5 + 12.7 * n + 7.0 * fill;
}
inline double pf_mx_us(const PfAttnPanel& p) {
    const int n_tiles = (p.M + PF_CHUNK - 1) / PF_CHUNK * p.grp, n_tg = (n_tiles + PF_MX_TILES - 1) / PF_MX_TILES;
    const int items = n_tg * p.Hkv, n_wg = std::min(p.wg_mx, items);
    auto item_us = [&](int it) { return pf_mx_item_us(p, n_tg - 1 - it / p.Hkv, n_tiles); };
    // the workgroup with the last group of tiles, and the one with the group before it (the last may have a row or two)
    double worst = 0.0;
    for (int first : {0, p.Hkv}) {
        double t = 0.0;
        for (int it = first; it < items; it += n_wg <= p.n_cu ? n_wg : items) t += item_us(it);
        worst = std::max(worst, t);
    }
    if (n_wg > p.n_cu) {   // more than a round: the rest start where the shortest of the first round have ended
        double all = 0.0;
        for (int tg = 0; tg < n_tg; ++tg) all += pf_mx_item_us(p, tg, n_tiles);
        worst = std::max(std::max(worst, item_us(p.n_cu - 1) + item_us(items - 1)), all * p.Hkv / p.n_cu);
    }
    return worst;
}
// The splits of which k_pf_attn's merge has room in LDS for one query's statistics: beyond them panels go to the other kernel,
// or, at the head_dims it has no instance for, the prompt goes through the 16-row forward.
constexpr int PF_VALU_MAX_SPLITS = 2560;
inline bool pf_panels_hold(int hd, int n) { return hd >= 64 || (n + PF_SPLIT - 1) / PF_SPLIT <= PF_VALU_MAX_SPLITS; }
inline bool pf_attn_on_matrix_cores(const PfAttnPanel& p) {
    if (p.wg_mx < 1) return false;
    return pf_chunk_splits(p, (p.M - 1) / PF_CHUNK) > PF_VALU_MAX_SPLITS || pf_mx_us(p) <= pf_valu_us(p);
}

// ---- the pipeline of k_pf_gemm<.., NT, .., JT, WJ>: what a wave has requested and not received when it waits.  Memory answers a
// wave in order, so a wait that lets n loads be on their way is over when all but the last n are here.  The waits below hold only
// if every load they count is issued: the kernel's last slabs, which request nothing, wait for everything instead.
constexpr int PF_STEPS = 4;   // steps of a slab: one weight load each per tile, and fragments of the pieces per column tile
constexpr int pf_weight_depth(int nt) { return nt == 1 ? 3 : (nt == 2 ? 2 : 1); }   // slabs of weights in a wave's registers
constexpr bool pf_one_ahead(int nt, int wj) { return wj == 1 && nt >= 3; }          // pieces one slab ahead, not two
// fragment = (piece * 4 + column tile) * 4 + step of a slab; wave w fetches fragments w, w + 8, .. of the column tiles it needs
constexpr bool pf_fetched(int jt, int fragment) { return ((fragment >> 2) & 3) < jt; }
constexpr int pf_min_fetch(int jt) { return jt == 4 ? 6 : (jt >= 2 ? 3 : 0); }      // of a slab, by every wave, at least
// Prologue: pieces of the first slab and its weights, pieces of the second (unless one ahead), the other slabs' weights.  What may
// be on its way when the first slab is read: everything behind its weights.
constexpr int pf_wait_first(int nt, int jt, int wj) {
    return pf_one_ahead(nt, wj) ? 0 : (pf_weight_depth(nt) - 1) * nt * PF_STEPS + pf_min_fetch(jt);
}
// A slab: pieces of the slab after the next one, then a weight load per step and tile.  What may be on its way when the next slab
// is read: this slab's requests and, with more than one slab of weights ahead, the weights requested behind the next slab's
// pieces (the prologue has as many).  One ahead: the pieces of the next slab come behind the first step, so the weights of the
// steps after it.
constexpr int pf_wait_slab(int nt, int jt, int wj) {
    return pf_one_ahead(nt, wj) ? nt * (PF_STEPS - 1) : (pf_weight_depth(nt) > 1 ? 2 : 1) * nt * PF_STEPS + pf_min_fetch(jt);
}

// ---- tiles and panels of the GEMMs.  A launch takes whole rounds of workgroups on the compute units, one each; its time in
// UNITS: one unit = a round of workgroups with one weight tile per wave over a reduction of 4096, 36 us.
constexpr int PF_SHARES = 8, PF_ROWS = 64;   // shares of the reduction dimension, prompt rows per workgroup tile

// A column (tile group and share group) and its my row tiles lie on one XCD, columns are dealt to the eight in turn: 36 columns
// of 7 row tiles are 252 workgroups, but 35 on some XCDs' 32 compute units, two rounds (d 2560, gate/up: 153 us; 6 row tiles 85).
inline double pf_rounds(int columns, int my, int n_cu) {
    const int per_xcd = (columns + 7) / 8 * my, cu = std::max(1, n_cu / 8);
    return (double)((per_xcd + cu - 1) / cu);
}
// QKV and gate/up with 8 nt tiles per workgroup (nt per wave; at nt < 3 twice as many and half the columns): smaller tiles read more
// bytes per matrix-core instruction (us per round, tile and reduction of 4096, d 4096 to 8192: 34-37 with three, 37-41 with two,
// 49-54 with one).
inline double pf_wide_units(int n_tiles, int my, int nt, int n_cu) {
    const double w[4] = {0.0, 1.4, 1.1, 1.0};
    return pf_rounds((n_tiles + 8 * nt - 1) / (8 * nt), my, n_cu) * nt * w[nt];
}
// 290 workgroups of 3 tiles are two rounds, 430 of 2 tiles two cheaper ones; 116 of 3 tiles fill half the chip, 172 of 2 tiles
// two thirds of it in two thirds of the time.
inline int pf_wide_tiles(int n_tiles, int my, int n_cu) {
    int best = 3;
    for (int nt = 2; nt >= 1; --nt)
        if (pf_wide_units(n_tiles, my, nt, n_cu) < pf_wide_units(n_tiles, my, best, n_cu) - 1e-9) best = nt;
    return best;
}
// O and down projection in tiles of 4 per wave: a tile's shares dealt to g workgroups, each with its prologue and its way out
// (a fifth of a share of 4096).  80 workgroups (5120 outputs, 512 rows): 4 groups are 320 workgroups of two shares, two rounds
// = 4.4 shares, 8 groups three rounds = 3.6.
inline double pf_narrow_shares(int n_nt, int my, int g, int n_cu) {
    return pf_rounds(n_nt * g, my, n_cu) * ((double)PF_SHARES / g + 0.2);
}
inline int pf_narrow_groups(int n_nt, int my, int n_cu) {
    int best = 1;
    for (int g = 2; g <= PF_SHARES; g *= 2)
        if (pf_narrow_shares(n_nt, my, g, n_cu) < pf_narrow_shares(n_nt, my, best, n_cu) - 1e-9) best = g;
    return best;
}
// A tile's shares dealt to workgroups of one-tile kernels (short panels; QKV is finished by a kernel of its own).
inline int pf_share_groups(int n_nt, int my, int n_cu) {
    int g = 1;
    while (g < PF_SHARES && n_nt * my * g < (n_cu * 3) / 4) g *= 2;
    return g;
}
// O and down: tiles of 4 per wave when they fill the chip, else of one (measured on the 7B shape: those win only below about 3/8
// of the compute units' worth of large tiles -- they read as many LDS bytes per matrix-core step as they feed it)
inline bool pf_tiles_fill(int n_tiles, int my, int n_cu) { return (n_tiles + 31) / 32 * my * PF_SHARES >= (n_cu * 3) / 8; }

struct PfModel {
    int d, hq, hkv, F, n_cu, hd;
    int max_tiles;     // row tiles of the largest panel that the workspace holds
    int wg_valu;       // workgroups k_pf_attn may use (regions of split partials)
    size_t mx_room;    // floats for the split partials of k_pf_attn_mx
};
// A panel of k_pf_attn_mx: split partials and their statistics of one workgroup, and the workgroups there is room for
constexpr size_t pf_mx_slot_floats(int hd, int n_splits) { return (size_t)n_splits * PF_MX_TILES * PF_CHUNK * (hd + 2); }
inline PfAttnPanel pf_attn_panel(const PfModel& m, int rows, int pos0) {
    PfAttnPanel p{m.hd, m.hkv / m.hd, m.hq / m.hkv, rows, pos0, m.n_cu, m.wg_valu, 0};
    if (m.hd < 64) return p;   // no instance
    const size_t slots = m.mx_room / pf_mx_slot_floats(m.hd, pf_chunk_splits(p, (rows - 1) / PF_CHUNK));
    const size_t items = (size_t)(((rows + PF_CHUNK - 1) / PF_CHUNK * p.grp + PF_MX_TILES - 1) / PF_MX_TILES) * p.Hkv;
    p.wg_mx = (int)std::min(items, slots);
    return p;
}
// A layer's time in us for a panel, from its kernels' times at 64 to 512 rows of eight shapes; over sixteen shapes, d 512 to 8192,
// it is 5 % off on average.
// A reduction takes whole blocks of 1024 values (d 2560 as long as 3072).  One block of one tile per wave: 8.6 us a round of
// workgroups (three tiles, d 4096: 103-115 us a round, 209-229 two), and 3 us a round for its prologue and way out.  What lies
// between the GEMMs: 20 us and the rows' way through memory.
constexpr double PF_BLOCK_US = 8.6, PF_ROUND_US = 3.0;
inline double pf_gemms_us(const PfModel& m, int my) {
    auto blocks = [](int K) { return (K + 1023) / 1024; };
    auto dealt = [&](int n_tiles, int K) {
        const int wgs = (n_tiles + 7) / 8, g = pf_share_groups(wgs, my, m.n_cu);
        return pf_rounds(wgs * g, my, m.n_cu) * (PF_SHARES / g) * 0.2 * PF_BLOCK_US * blocks(K) + 2 * PF_ROUND_US;
    };
    auto wide = [&](int n_tiles, int K) {
        const int nt = pf_wide_tiles(n_tiles, my, m.n_cu);
        return pf_wide_units(n_tiles, my, nt, m.n_cu) * PF_BLOCK_US * blocks(K) +
               pf_rounds((n_tiles + 8 * nt - 1) / (8 * nt), my, m.n_cu) * PF_ROUND_US;
    };
    auto narrow = [&](int K) {
        if (!pf_tiles_fill(m.d / 16, my, m.n_cu)) return dealt(m.d / 16, K);
        const int n_nt = (m.d / 16 + 31) / 32;
        return pf_narrow_shares(n_nt, my, pf_narrow_groups(n_nt, my, m.n_cu), m.n_cu) * 0.5 * PF_BLOCK_US * blocks(K) + PF_ROUND_US;
    };
    const int outs = m.hq + 2 * m.hkv, qkv_tiles = outs / 16;
    const bool qkv_dealt = pf_wide_tiles(qkv_tiles, my, m.n_cu) == 1 && pf_share_groups((qkv_tiles + 7) / 8, my, m.n_cu) > 1;
    return (qkv_dealt ? dealt(qkv_tiles, m.d) + 2 * PF_ROUND_US : wide(qkv_tiles, m.d)) + narrow(m.hq) + wide(m.F / 8, m.d) + narrow(m.F);
}
inline double pf_panel_us(const PfModel& m, int rows, int pos0, double gemms_us) {
    // of few rows one or two of the tile's four column tiles are multiplied
    const double few = rows <= 16 ? 0.8 : rows <= 32 ? 0.9 : 1.0;
    const PfAttnPanel p = pf_attn_panel(m, rows, pos0);
    const double mx = p.wg_mx > 0 ? pf_mx_us(p) : 1e300, valu = pf_valu_us(p);
    return few * gemms_us + std::min(mx, valu) + 20.0 + 1.1 * (rows / (double)PF_ROWS) * (m.d / 1024.0);
}
// The cut of `rows` rows from position pos0 into panels: full panels and a rest, unless the best cut is better by 2.5 % or more.  777
// rows of the 13B shape (4 layers) as 7 + 6 tiles and not 8 + 5: 6.66 -> 6.26 ms, gate/up in 2 + 2 rounds of workgroups and not
// 4 + 2; 1100 of the 7B shape as 2 + 8 + 8: 6.65 -> 6.28 (attention behind 8 splits costs a few rows what it costs a full panel).
// Over 20 shapes, d 512 to 8192, and 17 lengths from 513 to 4096 no cut that is chosen was slower than full panels, those that
// differ are 7 % quicker on average, 2 to 23 %; without attention and the XCDs in the model the same rule lost up to 23 % (d 2560, 3500 rows).
// Long prompts are cut PF_CUT_TILES row tiles at a time (the caller comes again with what is left): up to 70 us of host work, in
// front of the first panel, and beside the GPU's from then on.
constexpr int PF_CUT_TILES = 64;
struct PfCut { int n; int tiles[PF_CUT_TILES]; };
inline PfCut pf_cut(const PfModel& m, int rows, int pos0) {
    const int all = (rows + PF_ROWS - 1) / PF_ROWS, P = m.max_tiles;
    const int R = all <= PF_CUT_TILES ? all : PF_CUT_TILES / P * P;   // (P <= 8)
    PfCut c{0, {}};
    double gemms[PF_CUT_TILES + 1];
    for (int t = 1; t <= std::min(R, P); ++t) gemms[t] = pf_gemms_us(m, t);
    auto us = [&](int from, int t) {
        return pf_panel_us(m, std::min(t * PF_ROWS, rows - from * PF_ROWS), pos0 + from * PF_ROWS, gemms[t]);
    };
    double best[PF_CUT_TILES + 1] = {0.0}, plain = 0.0;
    int last[PF_CUT_TILES + 1] = {0};
    for (int r = 1; r <= R; ++r) {
        best[r] = 1e300;
        for (int t = std::min(r, P); t >= 1; --t) {
            const double v = best[r - t] + us(r - t, t);
            if (v < best[r] - 1e-9) { best[r] = v; last[r] = t; }
        }
    }
    for (int r = 0; r < R; r += P) plain += us(r, std::min(P, R - r));
    const bool other = best[R] <= 0.975 * plain;
    for (int r = R; r > 0; ++c.n) {   // from the end
        const int rest = R % P == 0 ? P : R % P, t = other ? last[r] : (c.n == 0 ? rest : P);
        c.tiles[c.n] = t;
        r -= t;
    }
    std::reverse(c.tiles, c.tiles + c.n);
    return c;
}

}  // namespace sdfp
