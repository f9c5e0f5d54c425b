// The cut of a prompt into panels, the tiles of its GEMMs and the counts of their pipeline, and which kernel runs a panel's
// attention (host arithmetic only).
#pragma once
#include <algorithm>

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
// UNITS: one unit = a round of workgroups with one weight tile per wave over a reduction of 4096, 38 us.
constexpr int PF_SHARES = 8, PF_ROWS = 64;   // shares of the reduction dimension, prompt rows per workgroup tile

inline double pf_rounds(int wgs, int n_cu) { return (double)((wgs + n_cu - 1) / n_cu); }
// QKV and gate/up with nt tiles per wave (and half the columns each at nt < 3): smaller tiles read more bytes per matrix-core
// instruction (measured per tile at 512 rows: 37.6 us with three, 39.8 with two; at a reduction of 8192 the ratio is 1.14).
inline double pf_wide_units(int n_tiles, int my, int nt, int n_cu) {
    const double w[4] = {0.0, 1.4, 1.1, 1.0};
    return pf_rounds((n_tiles + 8 * nt - 1) / (8 * nt) * my, n_cu) * nt * w[nt];
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
inline double pf_narrow_shares(int wgs, int g, int n_cu) { return pf_rounds(wgs * g, n_cu) * ((double)PF_SHARES / g + 0.2); }
inline int pf_narrow_groups(int wgs, int n_cu) {
    int best = 1;
    for (int g = 2; g <= PF_SHARES; g *= 2)
        if (pf_narrow_shares(wgs, g, n_cu) < pf_narrow_shares(wgs, best, n_cu) - 1e-9) best = g;
    return best;
}
struct PfModel { int d, hq, hkv, F, n_cu; };
// A layer's GEMMs over my row tiles, and half a unit for what a panel costs besides.
inline double pf_panel_units(const PfModel& m, int my) {
    const int qkv = (m.hq + 2 * m.hkv) / 16, gu = m.F / 8, out = (m.d + 511) / 512 * my;
    const double narrow = pf_narrow_shares(out, pf_narrow_groups(out, m.n_cu), m.n_cu) * 4.0 / PF_SHARES;
    return (pf_wide_units(qkv, my, pf_wide_tiles(qkv, my, m.n_cu), m.n_cu) + pf_wide_units(gu, my, pf_wide_tiles(gu, my, m.n_cu), m.n_cu)) *
               (m.d / 4096.0) + narrow * (m.hq + m.F) / 4096.0 + 0.5;
}
// Row tiles of the next panel of a prompt that has `rows` left, at most max_tiles (<= PF_CUT_TILES): a full panel or the rest, unless
// another cut of what is left is better by 3 % or more -- then its largest panel.  777 rows of the 13B shape: 7 + 6 tiles
// (gate/up in 2 + 2 rounds of workgroups) and not 8 + 5 (4 + 2): 72.1 -> 67.8 ms; 2000 rows 42.0 -> 38.6 of 8 layers.  Beyond PF_CUT_TILES tiles the size with the least time per tile.
constexpr int PF_CUT_TILES = 64;
inline int pf_next_panel(const PfModel& m, int rows, int max_tiles) {
    const int R = (rows + PF_ROWS - 1) / PF_ROWS, rest = rows - (R - 1) * PF_ROWS;
    double cost[PF_CUT_TILES + 1] = {0.0}, best[PF_CUT_TILES + 1] = {0.0};
    int largest[PF_CUT_TILES + 1] = {0}, even = max_tiles;
    for (int t = 1; t <= max_tiles; ++t) cost[t] = pf_panel_units(m, t);
    for (int t = 1; t < max_tiles; ++t)
        if (cost[t] / t < 0.97 * cost[max_tiles] / max_tiles && cost[t] / t < cost[even] / even) even = t;
    if (R > PF_CUT_TILES) return even;
    // a panel of one tile is the last one; of few rows it multiplies one or two of the tile's four column tiles (measured)
    best[1] = cost[1] * (rest <= 16 ? 0.8 : rest <= 32 ? 0.9 : 1.0);
    largest[1] = 1;
    for (int r = 2; r <= R; ++r) {
        best[r] = 1e300;
        for (int t = 1; t <= std::min(r, max_tiles); ++t)
            if (best[r - t] + cost[t] < best[r] - 1e-9) { best[r] = best[r - t] + cost[t]; largest[r] = std::max(t, largest[r - t]); }
    }
    const double plain = R / max_tiles * cost[max_tiles] + (R % max_tiles == 1 ? best[1] : cost[R % max_tiles]);
    return best[R] > 0.97 * plain ? std::min(R, max_tiles) : largest[R];
}

}  // namespace sdfp
