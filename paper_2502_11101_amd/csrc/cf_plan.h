// The launch plan of the 16-bit attention path: how rows, tokens and splits map to workgroups and where the partial results live in
// the workspace.  Host arithmetic on the call's sizes alone, free of device code, so that a host program can work a plan out.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "cachefocus.h"

namespace cf {
namespace attn {

constexpr int kWaves = 4;       // wavefronts of a group
constexpr int kD = 128;
constexpr int kTile = 32;       // tokens per tile
constexpr int kMaxSplit = 32;
constexpr int kRegEntries = 64; // the longest table that the attention kernels keep in registers
constexpr int kSoloWaves = 8;   // wavefronts of attn_solo_kernel's workgroups, each with tiles of its own

struct Plan {
    int group;          // query heads per kv head
    int row_blocks;     // 16-row blocks of the stacked rows of one kv head
    int wide;           // 0: attn_tile_kernel or attn_solo_kernel (few rows), 1: attn_wide_kernel, 2: its CAUSAL variant
    int nrb;            // 64-row passes of a workgroup's rows (what the combine kernel handles at a time)
    int rows_wg;        // rows a workgroup has room for: 64 * nrb
    int n_rg;           // row groups per (query, kv head)
    int blocks_rg;      // 16-row blocks per row group
    int units_per_b, units, nsplit, slots;
    int tile;           // tokens per tile: 32 (16 for fp32 tensors, cf_attn_plain.hip)
    int groups;         // runs of tiles per workgroup: 1 or 2 (groups of four wavefronts), kSoloWaves (attn_solo_kernel)
    int direct_out;     // one split: the attention kernel writes the output rows itself, nothing to merge
    size_t off_ml, off_opart, off_massml, off_masspart, total;
    size_t masspart_bytes;      // one layer's slot partials (the ledger holds CF_MAX_PENDING + 1 such parts)
};

// Tiles of a (query, kv head): every segment may end in a ragged one.
inline int64_t plan_tiles(int seg_stride, int64_t max_kv_tokens) { return max_kv_tokens / kTile + seg_stride; }

// Splits of a (query, kv head, row group): the CUs are shared out, each split has at least `least` tiles.
inline int plan_splits(int64_t units, int64_t tiles, int least) {
    return (int)std::max<int64_t>(std::min({256 / units, std::max<int64_t>(tiles / least, 1), (int64_t)kMaxSplit}), 1);
}

inline void plan_rows(Plan& p, int batch, int n_kv_heads, int n_rg, int nrb) {
    p.n_rg = n_rg;
    p.nrb = nrb;
    p.blocks_rg = (p.row_blocks + n_rg - 1) / n_rg;
    p.rows_wg = 64 * nrb;
    p.units_per_b = n_kv_heads * n_rg;
    p.units = batch * p.units_per_b;
}

// The partial results in the workspace.  A (segment, run of tiles) pair has slot segment + run: both only grow along the tile list.
// With one split nobody reads or writes the row statistics.  Their room stays: it is part of the bytes reported, and without it a workspace sized for
// many queries would no longer serve some smaller batches, which are split (513 of 82 593 such pairs of a sweep, 12 queries' for one among them).
inline void plan_layout(Plan& p, int seg_stride) {
    p.direct_out = p.nsplit == 1;
    p.slots = seg_stride + p.nsplit * p.groups;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
    p.off_ml = take((size_t)p.units * p.nsplit * p.rows_wg * 2 * sizeof(float));
    p.off_opart = take(p.direct_out ? 0 : (size_t)p.units * p.nsplit * p.rows_wg * kD * sizeof(uint16_t));
    p.off_massml = take((size_t)p.units * p.slots * p.rows_wg * 2 * sizeof(float));
    p.masspart_bytes = ((size_t)p.units * p.nrb * p.slots * sizeof(float) + 255) & ~(size_t)255;
    p.off_masspart = take(p.masspart_bytes * (CF_MAX_PENDING + 1));
    p.total = off;
}

// attn_tile_kernel's plan, for at most four row blocks.
inline Plan tile_plan(Plan p, int batch, int n_kv_heads, int seg_stride, int64_t max_kv_tokens) {
    // Few stacked rows (MHA-like, HBM-bound): one row block per wavefront, small tiles, so that ragged
    // segment ends waste little and a split still holds several tiles; two groups of four wavefronts per
    // workgroup run two tiles at a time on one CU and hide each other's LDS and barrier waits.
    plan_rows(p, batch, n_kv_heads, 1, 1);
    p.groups = 2;
    const int64_t tiles = plan_tiles(seg_stride, max_kv_tokens);
    // One launch wave: a CU holds one workgroup at a time (8 wavefronts of about 190 registers), so a grid a little past the 256
    // CUs runs two rounds, the second nearly empty, each with its prologue and tail.  Rounded down and
    // not up, calls that 256 does not divide measured: 6 decode queries x 32 heads over 1017-1573 tokens (192
    // units, two splits against one) 37.6 -> 26.5 us, 17 x 4 heads over 1355-1704 (68 units, four against three) 26.3 -> 19.0,
    // 28 x 2 heads over 723 (56 units) 18.6 -> 13.1, 3 layer queries x 32 heads, 7 short documents (96 units) 28.0 -> 22.2.
    // A split has about two tiles for each of the two groups.
    // The exception is a long batch that would leave over a quarter of the CUs idle: its halves even out unequal lengths, which the host
    // does not know, and cost less where the lengths are equal than they save where they are not.  Decode queries x 4 heads, one
    // split against two: up to 4096 tokens, lengths a fifth of that and more: 144 units 78 -> 64 us, 160 78 -> 62, 176 80 -> 74; up to
    // 12000: 198 -> 154, 204 -> 186, 207 -> 175; all of 4096: 82 -> 95, 82 -> 97, 83 -> 100.  At 192 units and more one is the better
    // (50 queries of 1000-5000 tokens, 200 units: 77 against 85), and for shorter lists (1024 tokens, 160 units: 31 against 35 and 39).
    const bool halves = p.units > 128 && p.units < 192 && tiles > 128;
    p.nsplit = halves ? 2 : plan_splits(p.units, tiles, 4);
    plan_layout(p, seg_stride);
    return p;
}

// attn_solo_kernel's, for one row block.
inline Plan solo_plan(Plan p, int seg_stride, int nsplit) {
    p.groups = kSoloWaves;
    p.nsplit = nsplit;
    plan_layout(p, seg_stride);
    return p;
}
constexpr int kSoloStride = 2, kSoloSplits = 8;      // the longest table and the most splits that get attn_solo_kernel

// attn_wide_kernel's, with row groups of up to `per_wave` blocks per wavefront and at most `groups` groups of wavefronts.
inline Plan wide_plan(Plan p, int batch, int n_kv_heads, int seg_stride, int64_t max_kv_tokens, int per_wave, int groups) {
    const int n_rg = (p.row_blocks + kWaves * per_wave - 1) / (kWaves * per_wave);
    const int nrb = ((p.row_blocks + n_rg - 1) / n_rg + kWaves - 1) / kWaves;
    plan_rows(p, batch, n_kv_heads, n_rg, nrb);
    const int64_t tiles = plan_tiles(seg_stride, max_kv_tokens);
    // four tiles a split are better than two: one query of 20 rows x 4 heads, ten documents, 23.5 us against 25.4
    p.nsplit = plan_splits(p.units, tiles, 4);
    // One group of wavefronts per workgroup for units past the CUs, two workgroups of which share one (30 documents x 32 heads, 960
    // units, encoded and stored: 84 us against 108 with two groups), and for splits of few tiles, which the second group's delay and the
    // merge of the groups cost more than it saves, the more the more blocks a wavefront has.  Around the lines, us with one group against
    // two, tiles a split in brackets.  Three blocks: layers of 64 queries x 2 heads, 384 rows, (10) 34.8 and 35.6, (12) 37.6 and 37.5,
    // (14) 39.5 and 39.0; 16 x 4, 336 rows, (11) 42.7 and 44.0, (13.5) 46.2 and 45.8; documents encoded x 2 heads, 12 of 228 tokens (10)
    // 28.6 and 30.3, of 300 (12) 33.3 and 34.7.  Two: 8 queries x 16 heads, 120 rows, (10.5) 37.3 and 37.7, 3 (11.4) 35.0 and 34.4; 4
    // documents x 32 heads of 228 (10) 28.6 and 30.0, x 4 heads of 260 (11) 26.1 and 25.5.  Five blocks, which leave one of the four
    // wavefronts idle and one half: 8 queries x 16 heads, 80 rows, (8) 29.3 and 30.4, (10) 36.1 and 35.7, 3 x 32 (10.5) 34.0 and 32.8.
    const int pays = p.blocks_rg <= 5 ? 10 : nrb == 2 ? 11 : 13;
    p.groups = groups == 2 && p.units <= 256 && tiles >= pays * p.nsplit ? 2 : 1;
    plan_layout(p, seg_stride);
    return p;
}
// (kv heads x row groups) is the second dimension of attn_wide_kernel's grid.
inline bool wide_grid_ok(int n_kv_heads, const Plan& p) { return (int64_t)n_kv_heads * p.n_rg <= 65535; }

inline Plan plan_shape(int n_q_heads, int n_kv_heads, int max_tq) {
    Plan p;
    p.group = n_q_heads / n_kv_heads;
    p.row_blocks = (p.group * max_tq + 15) / 16;
    p.wide = p.row_blocks > 4;
    p.tile = kTile;
    return p;
}

// The plan to fall back on for its workspace: no run of tiles beyond what fills the CUs, no row group beyond the fewest.  (Where more row
// groups do without splits, they take less still.)
inline Plan least_plan(int n_q_heads, int n_kv_heads, int batch, int max_tq, int seg_stride, int64_t max_kv_tokens) {
    const Plan p = plan_shape(n_q_heads, n_kv_heads, max_tq);
    return p.wide ? wide_plan(p, batch, n_kv_heads, seg_stride, max_kv_tokens, 3, 1) : tile_plan(p, batch, n_kv_heads, seg_stride, max_kv_tokens);
}

// The plan that the sizes of a call ask for.
inline Plan best_plan(int n_q_heads, int n_kv_heads, int batch, int max_tq, int seg_stride, int64_t max_kv_tokens) {
    const int64_t tiles = plan_tiles(seg_stride, max_kv_tokens);
    Plan p = plan_shape(n_q_heads, n_kv_heads, max_tq);
    if (p.wide) {
        // Many rows (GQA, long queries): row groups of up to three blocks per wavefront, or of up to two.  Fewer groups stage the same keys
        // less often, but three blocks keep every register busy and two do not: a tile's time goes about as 4 * blocks per wavefront
        // + 2 (each about 0.09 us for one group of wavefronts), and what it adds up to depends on how the units fill the CUs.  448
        // rows, 4 kv heads, as four groups of two blocks against three of three: one query of 50 documents 37.8 us against 41.7, 8 queries
        // of 20 66 against 76, 32 171 against 197.  384 rows, 64 queries x 2 kv heads, as three of two 168 us, as two of three 127 (384
        // units against 256); five documents of 100-200 tokens x 7 rows, 4 kv heads, 22.7 against 24.8 (220 units against 140).  Past the CUs a share of a round costs most of one: 107 rows x 6, 36
        // queries x 2 heads, 10 documents, as four of three (288 units) 91 us, as six of two (432) 80; 83 rows x 7, 14 queries x 4 heads, 10
        // documents, as five of two (280) 95, as four of three (224) 76; 129 rows x 6, 41 queries x 2 heads, as seven of two (574) 91, as
        // five of three (410) 75.  Splits pay for their partial rows, written and read, and for the merge: about 30 of those parts per 64
        // rows of every CU (8 us for three blocks).  12 documents of 160 tokens x 2 heads, encoded, as five of three in two splits 32.9
        // us, as eight of two in one 20.5; 8 of 228 35.9 and 23.8; 15 queries x 4 heads, 336 rows, 7 documents of 67 46.4 and 40.5.
        const Plan three = wide_plan(p, batch, n_kv_heads, seg_stride, max_kv_tokens, 3, 2);
        const Plan two = wide_plan(p, batch, n_kv_heads, seg_stride, max_kv_tokens, 2, 2);
        // past the CUs two workgroups share one, at 1.7 times what one alone takes, and a third begins when they end
        auto cost = [tiles](const Plan& c) {
            const double rounds = c.units > 512 ? std::max(c.units / 256., 2.7) : 1.7;
            const double merge = c.nsplit > 1 ? 30. * c.nrb * c.units * c.nsplit / 256 : 0;
            return (4 * c.nrb + 2) * tiles * (c.units > 256 ? rounds : 1. / c.nsplit) + merge;
        };
        return wide_grid_ok(n_kv_heads, two) && cost(two) < cost(three) ? two : three;
    }
    p = tile_plan(p, batch, n_kv_heads, seg_stride, max_kv_tokens);
    // attn_solo_kernel: one row block over at most two table entries (a decode step: the cache and the own block; short documents over
    // the prefix) and at most eight splits.  Longer tables are layer calls, which ask for masses: statistics of eight wavefronts per
    // segment to reduce cost more than the attention saves (10 documents of 160 tokens x 12 rows x 32 heads 24.8 us against 23.2 with
    // attn_tile_kernel, 30 documents x 16 rows 33.9 against 31.3).  The line does not ask for masses, so that a call's outputs do not
    // depend on whether it wants them.
    const int ns = p.nsplit;
    if (p.row_blocks > 1 || seg_stride > kSoloStride || ns > kSoloSplits) return p;
    // Past four rounds of the CUs the merge of eight wavefronts per workgroup costs what their streams save: 2048 units of ten tiles 84.0
    // us against 78.8 with attn_tile_kernel, of 22 135.0 and 134.1; 1024 of ten 43.9 and 43.2, of 48 136.5 and 136.7.
    if (p.units > 1024) return p;
    // Lists of up to two tiles per wavefront, which are all in flight at once, take one split and no merge: one conversation of 200 | 400
    // tokens x 32 heads 10.6 -> 8.4 | 11.2 -> 10.0 us, 32 of 200 | 400 x 4 heads 15.2 -> 9.2 | 17.3 -> 12.1.  Where the CUs allow two
    // splits at most, lists of up to four tiles per wavefront do: 4 conversations of 881 tokens x 32 heads 21.8 -> 17.8, of 150-880 19.9
    // -> 16.0; of 3000 40.7 would be 43.4.
    if (tiles <= 2 * kSoloWaves || (p.units > 85 && tiles <= 4 * kSoloWaves)) return solo_plan(p, seg_stride, 1);
    // One split: 40 conversations of 1000-2000 tokens x 4 heads 32.1 us against 33.7, 28 of 850-2100 x 8 39.0 against 40.0.  (Equal lists
    // just past two tiles per wavefront are up to 4.5 % slower, unequal ones faster; the host does not know.)
    if (ns == 1) return solo_plan(p, seg_stride, 1);
    // Two: from 112 units on, equal lists within 2 % either way and unequal ones faster, below, equal ones are slower.  x 4 heads, us
    // against attn_tile_kernel, 1972 tokens | 2500 | 1000-4000: 22 conversations 27.9 and 26.9 | 31.9 and 30.5 | 38.0 and 39.4; 25 30.1 and
    // 29.5 | 34.3 and 33.8 | 40.5 and 41.1; 28 32.1 and 31.8 | 36.3 and 36.3 | 42.5 and 43.1; 32 34.7 and 34.3 | 39.5 and 40.1 | 45.9 and 47.0.
    if (ns == 2) return p.units > 112 ? solo_plan(p, seg_stride, 2) : p;
    // More: of up to four tiles (one conversation of 881 tokens x 32 heads in seven 11.9 us, with attn_tile_kernel 12.6; in one, two, three
    // and four splits 14.6, 13.9, 13.2 and 12.4); longer ones are the better there (1500 tokens 15.3 and 14.5, two of them
    // 20.7 and 18.7, 8 of 1000-2000 x 4 heads 16.0 and 15.2), as are those of more than eight splits, which it spreads over more CUs (4
    // units x 2000 tokens 12.7 us as eight splits here, 12.2 as 16 there, x 14000 30.4 and 20.3).
    return tiles < 5 * ns ? solo_plan(p, seg_stride, ns) : p;
}

// What cf_prefill_workspace_bytes reports: no plan of these arguments takes more, nor one of a smaller max_kv_tokens or seg_stride, so that
// a workspace for the longest lists serves all shorter ones.  Every kernel's own splits, groups and slots grow with both
// arguments; the plan goes from kernel to kernel and back, so it is the most that any of them takes up to here.  A call whose least plan fits
// the buffer of the entry point that brings its own never takes more than that.  Many rows count at least as full row groups of twelve
// blocks with a split for every two tiles, so that a workspace for longer queries serves shorter ones as far as their splits allow.
inline size_t workspace_bytes(int n_q_heads, int n_kv_heads, int batch, int max_tq, int seg_stride, int64_t max_kv_tokens) {
    const Plan p = plan_shape(n_q_heads, n_kv_heads, max_tq);
    const Plan least = least_plan(n_q_heads, n_kv_heads, batch, max_tq, seg_stride, max_kv_tokens);
    size_t most = least.total, full = 0;
    if (p.wide) {
        const Plan two = wide_plan(p, batch, n_kv_heads, seg_stride, max_kv_tokens, 2, 2);
        most = std::max(most, wide_plan(p, batch, n_kv_heads, seg_stride, max_kv_tokens, 3, 2).total);
        if (wide_grid_ok(n_kv_heads, two)) most = std::max(most, two.total);
        Plan f = least;
        plan_rows(f, batch, n_kv_heads, least.n_rg, 3);
        f.nsplit = plan_splits(f.units, plan_tiles(seg_stride, max_kv_tokens), 2);
        plan_layout(f, seg_stride);
        full = f.total;
    } else if (p.row_blocks == 1) {
        const int stride = std::min(seg_stride, kSoloStride);
        const Plan tile = tile_plan(p, batch, n_kv_heads, stride, max_kv_tokens);
        most = std::max(most, solo_plan(tile, stride, std::min(tile.nsplit, kSoloSplits)).total);
    }
    return std::max(least.total <= CF_STATIC_SCRATCH_BYTES ? std::min(most, CF_STATIC_SCRATCH_BYTES) : most, full);
}

// attn_wide_kernel's CAUSAL variant: one split and one group of wavefronts, wherever there are several row groups, whose lists then end at
// different tokens of the own block, and for own blocks of half the list and more (a document's encoding over the prefix).  28 heads over 4, us
// without and with it: 40 queries of 130 tokens over 182 | 272 | 532 others 74.8 and 68.4 | 80.3 and 73.2 | 116.6 and 108.0; 32 of 64 over 1532
// 95.6 and 91.6, over 3032 156.6 and 156.4; 32 heads, 6 of 400 over 1632 170.7 and 164.3.  One row group, 30 documents x 32 heads encoded (the own
// block's share in brackets): of 160 tokens (0.83) 72.9 and 71.2, of 135 (0.58) 72.1 and 68.4, of 128 (0.57) 62.4 and 62.3, of 96 (0.50) 49.6 and
// 49.1; 50 x 16 heads over 8 of 70 (0.67) 25.8 and 24.7.  Around the line layers, with masses, differ by up to 2 % either way: 24 queries of 192
// tokens x 16 heads (0.60) 39.3 and 38.8, (0.52) 43.9 and 44.7, (0.46) 44.8 and 45.7, (0.40) 48.3 and 48.9; of 128 (0.67) 25.7 and 25.9, (0.50)
// 29.6 and 29.9, (0.36) 32.1 and 32.6.  Far below it there are few tiles to leave out.
inline bool causal_pays(const Plan& p, int max_tq, int seg_stride, int64_t max_kv_tokens) {
    return p.wide && p.nsplit == 1 && p.groups == 1 && seg_stride <= kRegEntries && (p.n_rg > 1 || 2 * (int64_t)max_tq >= max_kv_tokens);
}

// `given`: the bytes of the call's workspace.  With as many as workspace_bytes reports the plan follows from the sizes alone; with fewer
// (sized for another batch, say) a call goes without the runs and row groups that do not fit.
inline Plan make_plan(int n_q_heads, int n_kv_heads, int batch, int max_tq, int seg_stride, int64_t max_kv_tokens, size_t given) {
    Plan p = best_plan(n_q_heads, n_kv_heads, batch, max_tq, seg_stride, max_kv_tokens);
    if (p.total > std::min(given, CF_STATIC_SCRATCH_BYTES)) {
        const Plan least = least_plan(n_q_heads, n_kv_heads, batch, max_tq, seg_stride, max_kv_tokens);
        if (p.total > given || least.total <= CF_STATIC_SCRATCH_BYTES) p = least;
    }
    if (causal_pays(p, max_tq, seg_stride, max_kv_tokens)) p.wide = 2;
    return p;
}

}  // namespace attn
}  // namespace cf
