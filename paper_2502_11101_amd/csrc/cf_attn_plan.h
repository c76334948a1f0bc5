// Shared by the 16-bit attention kernels and the kernels that reduce their partial results: the launch plan
// (how rows, tokens and splits map to workgroups and where the partials live in the workspace), the per-query
// segment table in its two forms (LDS, registers) with the tile walk over it, and the MFMA wrappers.
#pragma once

#include <algorithm>

#include "cf_common.h"
#include "cf_select_dev.h"

namespace cf {
namespace attn {

constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int kD = 128;
constexpr int kHalf = 64;
constexpr int kKRow = 272;      // bytes per token of a staged K tile
constexpr int kMaxSegs = 256;
constexpr int kMaxSplit = 32;
constexpr int kSoloWaves = 8;   // wavefronts of attn_solo_kernel's workgroups, each with tiles of its own
constexpr int kMaxSub = 2 * kMaxSplit;       // runs of tiles of a (query, kv head, row group): splits x groups

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

struct Plan {
    int group;          // query heads per kv head
    int row_blocks;     // 16-row blocks of the stacked rows of one kv head
    int wide;           // 0: attn_tile_kernel or attn_solo_kernel (few rows), 1: attn_wide_kernel
    int nrb;            // 64-row passes of a workgroup's rows (what the combine kernel handles at a time)
    int rows_wg;        // rows a workgroup has room for: 64 * nrb
    int n_rg;           // row groups per (query, kv head)
    int blocks_rg;      // 16-row blocks per row group
    int units_per_b, units, nsplit, slots;
    int tile;           // tokens per tile: 32 or 64
    int groups;         // runs of tiles per workgroup: 1 or 2 (groups of four wavefronts), kSoloWaves (attn_solo_kernel)
    int direct_out;     // one split: the attention kernel writes the output rows itself, nothing to merge
    size_t off_ml, off_opart, off_massml, off_masspart, total;
    size_t masspart_bytes;      // one layer's slot partials (the ledger holds kMaxPending + 1 such parts)
};

// `small`: the fewest row groups and runs (see make_plan).
inline Plan plan_of(int n_q_heads, int n_kv_heads, int batch, int max_tq, int seg_stride, int64_t max_kv_tokens, bool small) {
    Plan p;
    const int group = n_q_heads / n_kv_heads;
    const int row_blocks = (group * max_tq + 15) / 16;
    p.group = group;
    p.row_blocks = row_blocks;
    const int64_t est_tiles = max_kv_tokens / 32 + seg_stride;           // every plan's tiles are of 32 tokens
    // splits of a (query, kv head, row group): the CUs are shared out, and a split of attn_tile_kernel has about two tiles for each of
    // its two groups (four a split are the better for attn_wide_kernel too: one query of 20 rows x 4 heads, ten documents, 23.5 us
    // against 25.4 with two)
    auto splits_of = [&](int64_t units) {
        const int64_t cap = std::max<int64_t>(est_tiles / 4, 1);
        return std::max<int64_t>(std::min({256 / units, cap, (int64_t)kMaxSplit}), 1);
    };
    if (row_blocks <= 4) {
        // Few stacked rows (MHA-like, HBM-bound): one row block per wavefront, small tiles, so that ragged
        // segment ends waste little and a split still holds several tiles; two groups of four wavefronts per
        // workgroup run two tiles at a time on one CU and hide each other's LDS and barrier waits.
        p.wide = 0;
        p.n_rg = 1;
        p.nrb = 1;
        p.tile = 32;
        p.groups = 2;
    } else {
        // Many rows (GQA, long queries): row groups of up to three blocks per wavefront, or of up to two.  Fewer groups stage the same keys
        // less often, but three blocks keep every register busy and two do not: a tile's time goes about as 4 * blocks per wavefront
        // + 2, and what it adds up to depends on how the units fill the CUs.  448 rows, 4 kv heads, as four groups of two blocks against
        // three of three: one query of 50 documents 37.8 us against 41.7, 8 queries of 20 66 against 76, 32 171 against 197.  384 rows, 64
        // queries x 2 kv heads, as three of two 168 us, as two of three 127 (384 units against 256); five documents of 100-200 tokens x 7
        // rows, 4 kv heads, 22.7 against 24.8 (220 units against 140).  Past the CUs a share of a round costs most of one: 107 rows x 6, 36
        // queries x 2 heads, 10 documents, as four of three (288 units) 91 us, as six of two (432) 80; 83 rows x 7, 14 queries x 4 heads, 10
        // documents, as five of two (280) 95, as four of three (224) 76; 129 rows x 6, 41 queries x 2 heads, as seven of two (574) 91, as
        // five of three (410) 75.
        p.wide = 1;
        p.tile = 32;
        double best = 0;
        for (int per_wave = 3; per_wave >= (small ? 3 : 2); --per_wave) {
            const int n_rg = (row_blocks + kWaves * per_wave - 1) / (kWaves * per_wave);
            const int nrb = ((row_blocks + n_rg - 1) / n_rg + kWaves - 1) / kWaves;
            if (per_wave < 3 && (int64_t)n_kv_heads * n_rg + 1 > 65535) continue;        // past the grid: fewer groups are taken instead
            const int64_t units = (int64_t)batch * n_kv_heads * n_rg;
            // past the CUs two workgroups share one, at 1.7 times what one alone takes, and a third begins when they end
            const double rounds = units > 512 ? std::max(units / 256., 2.7) : 1.7;
            const double cost = (4 * nrb + 2) * (units > 256 ? rounds : 1. / splits_of(units));
            if (per_wave == 3 || cost < best) { best = cost; p.n_rg = n_rg; p.nrb = nrb; }
        }
    }
    p.blocks_rg = (row_blocks + p.n_rg - 1) / p.n_rg;
    p.rows_wg = 64 * p.nrb;
    p.units_per_b = n_kv_heads * p.n_rg;
    p.units = batch * p.units_per_b;
    // One launch wave: a CU holds one workgroup of either kernel at a time (8 wavefronts of about 190 and 250 registers), so a
    // grid a little past the 256 CUs runs two rounds, the second nearly empty, each with its prologue and tail.  Rounded down and
    // not up, attn_tile_kernel's calls that 256 does not divide measured: 6 decode queries x 32 heads over 1017-1573 tokens (192
    // units, two splits against one) 37.6 -> 26.5 us, 17 x 4 heads over 1355-1704 (68 units, four against three) 26.3 -> 19.0,
    // 28 x 2 heads over 723 (56 units) 18.6 -> 13.1, 3 layer queries x 32 heads, 7 short documents (96 units) 28.0 -> 22.2.
    // The exception is a long batch that would leave over a quarter of the CUs idle: its halves even out unequal lengths, which the host
    // does not know, and cost less where the lengths are equal than they save where they are not.  Decode queries x 4 heads, one
    // split against two: up to 4096 tokens, lengths a fifth of that and more: 144 units 78 -> 64 us, 160 78 -> 62, 176 80 -> 74; up to
    // 12000: 198 -> 154, 204 -> 186, 207 -> 175; all of 4096: 82 -> 95, 82 -> 97, 83 -> 100.  At 192 units and more one is the better
    // (50 queries of 1000-5000 tokens, 200 units: 77 against 85), and for shorter lists (1024 tokens, 160 units: 31 against 35 and 39).
    const bool halves = !p.wide && p.units > 128 && p.units < 192 && est_tiles > 128;
    int64_t ns = halves ? 2 : splits_of(p.units);
    // attn_solo_kernel: one row block over at most two table entries (a decode step: the cache and the own block; short documents over
    // the prefix) and at most eight splits, as many runs of tiles as the reductions have room for.  Longer tables are layer calls, which ask
    // for masses: eight statistics per segment and split to reduce cost more than the attention saves (10 documents of 160 tokens x 12
    // rows x 32 heads 24.8 us against 23.2 with attn_tile_kernel, 30 documents x 16 rows 33.9 against 31.3).  More splits are long lists
    // over few units, which attn_tile_kernel spreads over more CUs (4 units x 2000 tokens 12.7 us as eight splits here, 12.2 as 16 there, x
    // 14000 30.4 and 20.3).  The line does not ask for masses, so that a call's outputs do not depend on whether it wants them.
    // Lists of up to two tiles per wavefront, which are all in flight at once, take one split and no merge: one conversation of 200 | 400
    // tokens x 32 heads 10.6 -> 8.4 | 11.2 -> 10.0 us, 32 of 200 | 400 x 4 heads 15.2 -> 9.2 | 17.3 -> 12.1; of 881 (seven splits) 13.5
    // would be 16.6.  Where the CUs allow two splits at most, lists of up to four tiles per wavefront do: 4 conversations of 881 tokens x 32
    // heads 21.8 -> 17.8, of 150-880 19.9 -> 16.0; of 3000 40.7 would be 43.4.
    // With more than two splits of more than four tiles attn_tile_kernel is the faster: 2 conversations of 1500 tokens x 32 heads 18.7 us
    // against 20.7, 1 14.5 against 15.3, 8 of 1000-2000 x 4 heads 15.2 against 16.0; with two up to 112
    // units 28.3 against 28.5 (3 of 1972 x 32) and 26.7 against 26.9 (28 of 1500 x 4), at 128 54.7 against 53.7 (32 of 1000-5000 x 4); with one 33.7 against 32.1 (40 of 1000-2000 x 4); with seven of four tiles 12.6 against 11.7.
    const bool whole = est_tiles <= 2 * kSoloWaves || (p.units > 85 && est_tiles <= 4 * kSoloWaves);
    const bool solo = !small && row_blocks == 1 && seg_stride <= 2 && ns <= kMaxSub / kSoloWaves && (whole || ns == 1 || (ns == 2 && p.units > 112) || est_tiles < 5 * ns);
    if (solo && whole) ns = 1;
    p.nsplit = (int)ns;
    p.direct_out = p.nsplit == 1;
    // attn_wide_kernel as one group of wavefronts per workgroup: for units past the CUs, two workgroups of which share one (30
    // documents x 32 heads, 960 units, encoded and stored: 84 us against 108 with two groups), and for splits of few tiles, which the second
    // group's delay and the merge of the groups cost more than it saves.  Around the line, us with one group against two: one query x 2
    // kv heads, 384 rows, under four tiles a split 29.0 against 32.0, 4 queries x 4 heads, 140 rows, seven 31.3 against 33.2; 8 queries x
    // 2 heads, 384 rows, fifteen 42.2 against 41.2, 2 x 32 heads, 130 rows, twelve 40.9 against 38.9.
    if (p.wide) p.groups = !small && p.units <= 256 && est_tiles >= 10 * ns ? 2 : 1;
    else if (solo) p.groups = kSoloWaves;
    p.slots = seg_stride + p.nsplit * p.groups;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
    p.off_ml = take((size_t)p.units * p.nsplit * p.rows_wg * sizeof(float2));
    p.off_opart = take(p.direct_out ? 0 : (size_t)p.units * p.nsplit * p.rows_wg * kD * sizeof(uint16_t));
    p.off_massml = take((size_t)p.units * p.slots * p.rows_wg * sizeof(float2));
    p.masspart_bytes = ((size_t)p.units * p.nrb * p.slots * sizeof(float) + 255) & ~(size_t)255;
    p.off_masspart = take(p.masspart_bytes * (kMaxPending + 1));
    p.total = off;
    return p;
}

// More row groups and more runs of tiles per workgroup take workspace.  Where that alone would carry a plan past the buffer of the entry
// point that brings its own, the plan does without.
inline Plan make_plan(int n_q_heads, int n_kv_heads, int batch, int max_tq, int seg_stride, int64_t max_kv_tokens) {
    const Plan p = plan_of(n_q_heads, n_kv_heads, batch, max_tq, seg_stride, max_kv_tokens, false);
    if (p.total <= CF_STATIC_SCRATCH_BYTES) return p;
    const Plan least = plan_of(n_q_heads, n_kv_heads, batch, max_tq, seg_stride, max_kv_tokens, true);
    return least.total <= CF_STATIC_SCRATCH_BYTES ? least : p;
}

// Per-query segment table in LDS with the tile prefix that defines the partition.
struct SegTable {
    int64_t tok[kMaxSegs];      // first token in its tensor
    int32_t vis[kMaxSegs];      // visible tokens (0 for a rejected entry)
    int32_t delta[kMaxSegs];    // relative shift: (new - stored) - (q_new - q_stored)
    int32_t self[kMaxSegs];     // 1 for the causal own block
    int32_t doc[kMaxSegs];      // document slot of the entry (-1: none)
    int32_t tile0[kMaxSegs + 1];// exclusive prefix of tile counts
    int32_t n;
};

// Per-query scalars and this thread's segment-table entry, fetched in one batch: the entry is
// read for the whole stride so that its load does not wait for the segment count.
struct QueryHead {
    int q0, tq_raw, n_seg, qdelta, q_new;
    int64_t q_total;
    cf_segment seg;
};

// `entry`: which table entry this thread takes (its index in the workgroup for the LDS table, its lane
// for the register table).
// Threads past the stride re-read the last entry instead of skipping the load — a conditional load makes
// the compiler wait for it inside the branch, before the scalar loads below are even issued (a whole round trip).
__device__ __forceinline__ QueryHead load_query_head(const AttnArgs& a, int b, int entry) {   // b: wave-uniform
    QueryHead h;
    h.seg = a.segs[(int64_t)b * a.seg_stride + min(entry, a.seg_stride - 1)];   // seg_stride >= 1; callers test entry < n
    const int q0 = a.q_off[b], q1 = a.q_off[b + 1], qt = a.q_off[a.batch], n = a.n_seg[b], qn = a.q_new_start[b];
    asm volatile("" ::"s"(q0), "s"(q1), "s"(qt), "s"(n), "s"(qn));    // all five scalar loads are out before any is used
    h.q0 = q0;
    h.tq_raw = q1 - q0;
    h.q_total = qt;
    h.n_seg = n;
    h.qdelta = qn - a.q_stored_start;
    h.q_new = qn;
    return h;
}

// All threads of a workgroup call this; every workgroup of query b builds the same table.
__device__ __forceinline__ void build_table(const AttnArgs& a, const QueryHead& h, SegTable* t, int tile_tokens) {
    const int tid = threadIdx.x;
    const cf_segment& seg = h.seg;
    int n = h.n_seg;
    if (n < 0 || n > a.seg_stride) {
        if (tid == 0) raise_flag(a.dev_flag, CF_FLAG_BAD_SEGMENT);
        n = n < 0 ? 0 : a.seg_stride;
    }
    const int tq = min(h.tq_raw, a.max_tq);
    // a query placed (or stored) outside the positional range attends nothing: every entry counts as empty
    const bool q_ok = positions_ok(h.q_new, tq, a.max_positions) && positions_ok(a.q_stored_start, tq, a.max_positions);
    if (!q_ok && tid == 0) raise_flag(a.dev_flag, CF_FLAG_POS_RANGE);
    if (tid < n) {
        const bool self = seg.kind == CF_SEG_SELF;
        const int64_t limit = self ? h.q_total : a.n_store_tokens;
        const bool bad = seg.kind < 0 || seg.kind > CF_SEG_SELF || seg.len < 0 || seg.tok_offset < 0 ||
                         seg.tok_offset + seg.len > limit || (self && a.k_self == nullptr);
        if (bad) raise_flag(a.dev_flag, CF_FLAG_BAD_SEGMENT);
        const int len_vis = bad ? 0 : (self ? min(seg.len, tq) : seg.len);
        const bool off_range = !(positions_ok(seg.new_start, len_vis, a.max_positions) &&
                                 positions_ok(seg.stored_start, len_vis, a.max_positions));
        if (off_range && !bad) raise_flag(a.dev_flag, CF_FLAG_POS_RANGE);
        const int vis = off_range || !q_ok ? 0 : len_vis;
        t->tok[tid] = seg.tok_offset;
        t->vis[tid] = vis;
        t->delta[tid] = seg.new_start - seg.stored_start - h.qdelta;
        t->self[tid] = self ? 1 : 0;
        t->doc[tid] = seg.doc;
        t->tile0[tid + 1] = (vis + tile_tokens - 1) / tile_tokens;
    }
    if (tid == 0) { t->n = n; t->tile0[0] = 0; }
    __syncthreads();
    if (tid < kWave) {                               // inclusive scan by the first wavefront
        int carry = 0;
        for (int c0 = 0; c0 < n; c0 += kWave) {
            const int s = c0 + tid;
            int v = s < n ? t->tile0[s + 1] : 0;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const int u = __shfl_up(v, o);
                if (tid >= o) v += u;
            }
            if (s < n) t->tile0[s + 1] = v + carry;
            carry += __shfl(v, kWave - 1);
        }
    }
    __syncthreads();
}

// split i of a list of `total` tiles owns [total*i/nsplit, total*(i+1)/nsplit)
__device__ __forceinline__ int split_begin(unsigned total, unsigned nsplit, unsigned i) { return (int)div_exact(total * i, nsplit); }
// the split that owns tile x
__device__ __forceinline__ int split_of(unsigned total, unsigned nsplit, unsigned x) { return (int)div_exact((x + 1) * nsplit - 1, total); }

template <int DT> struct Mma;
template <> struct Mma<CF_BF16> {
    static __device__ __forceinline__ f32x4 run(uint4 a, uint4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
    static __device__ __forceinline__ float lo(uint32_t w) { return __uint_as_float(w << 16); }
    static __device__ __forceinline__ float hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
    static __device__ __forceinline__ uint32_t pack(float x, float y) {
        f32x2 v = {x, y};
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    }
};
template <> struct Mma<CF_F16> {
    static __device__ __forceinline__ f32x4 run(uint4 a, uint4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
    static __device__ __forceinline__ float lo(uint32_t w) { return (float)__builtin_bit_cast(f16x2, w)[0]; }
    static __device__ __forceinline__ float hi(uint32_t w) { return (float)__builtin_bit_cast(f16x2, w)[1]; }
    static __device__ __forceinline__ uint32_t pack(float x, float y) {
        f32x2 v = {x, y};
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
    }
};

// One tile of the walk over a split's tiles; ntok == 0 marks "no tile left".
struct Tile { int seg, tok0, ntok, delta, self; };

// The same table for at most 64 segments, held in registers: lane s of every wavefront describes segment s.
// Built by each wavefront for itself — no LDS, no barrier — and searched with a ballot and lane reads.
struct RegSegTable {
    int64_t tok;                // this lane's segment, as in SegTable
    int32_t vis, delta, self;
    int32_t t0, t1;             // its tiles [t0, t1)
    int32_t n, total;           // wavefront-uniform: segments, tiles
};

// `h.seg` is entry `lane`; seg_stride <= 64.
__device__ __forceinline__ RegSegTable build_reg_table(const AttnArgs& a, const QueryHead& h, int lane, int tile_tokens) {
    RegSegTable t;
    const cf_segment& seg = h.seg;
    int n = h.n_seg;
    if (n < 0 || n > a.seg_stride) {
        if (lane == 0) raise_flag(a.dev_flag, CF_FLAG_BAD_SEGMENT);
        n = n < 0 ? 0 : a.seg_stride;
    }
    const int tq = min(h.tq_raw, a.max_tq);
    // a query placed (or stored) outside the positional range attends nothing: every entry counts as empty
    const bool q_ok = positions_ok(h.q_new, tq, a.max_positions) && positions_ok(a.q_stored_start, tq, a.max_positions);
    if (!q_ok && lane == 0) raise_flag(a.dev_flag, CF_FLAG_POS_RANGE);
    int vis = 0;
    t.tok = 0; t.delta = 0; t.self = 0;
    if (lane < n) {
        const bool self = seg.kind == CF_SEG_SELF;
        const int64_t limit = self ? h.q_total : a.n_store_tokens;
        const bool bad = seg.kind < 0 || seg.kind > CF_SEG_SELF || seg.len < 0 || seg.tok_offset < 0 ||
                         seg.tok_offset + seg.len > limit || (self && a.k_self == nullptr);
        if (bad) raise_flag(a.dev_flag, CF_FLAG_BAD_SEGMENT);
        const int len_vis = bad ? 0 : (self ? min(seg.len, tq) : seg.len);
        const bool off_range = !(positions_ok(seg.new_start, len_vis, a.max_positions) &&
                                 positions_ok(seg.stored_start, len_vis, a.max_positions));
        if (off_range && !bad) raise_flag(a.dev_flag, CF_FLAG_POS_RANGE);
        vis = off_range || !q_ok ? 0 : len_vis;
        t.tok = seg.tok_offset;
        t.delta = seg.new_start - seg.stored_start - h.qdelta;
        t.self = self ? 1 : 0;
    }
    t.vis = vis;
    const int tiles = (vis + tile_tokens - 1) / tile_tokens;
    t.t1 = wave_inclusive_scan(tiles);
    t.t0 = t.t1 - tiles;
    t.n = n;
    t.total = __builtin_amdgcn_readlane(t.t1, kWave - 1);
    return t;
}

// The segment that owns tile x (x < total) and its fields, in scalars.  `prev`: the segment found last (-1: none).
struct FoundSegment { int seg, first, end, vis, delta, self; int64_t tok; };

__device__ __forceinline__ FoundSegment find_segment(const SegTable& tbl, int x, int lane, int prev) {
    // the first segment whose tiles reach past x: every lane tests one entry per round
    int s = 0;
    for (int s0 = prev < 0 ? 0 : (prev & ~(kWave - 1));; s0 += kWave) {
        const int idx = s0 + lane;
        const unsigned long long hit = __ballot(idx < tbl.n && tbl.tile0[idx + 1] > x);
        if (hit) { s = s0 + __builtin_ctzll(hit); break; }
    }
    // (the values are the same in every lane; taking them from the first one tells the compiler so, which keeps
    // everything derived from them — tile descriptions, base addresses — on the scalar unit)
    FoundSegment f;
    f.seg = s;
    f.first = __builtin_amdgcn_readfirstlane(tbl.tile0[s]);
    f.end = __builtin_amdgcn_readfirstlane(tbl.tile0[s + 1]);
    f.vis = __builtin_amdgcn_readfirstlane(tbl.vis[s]);
    f.delta = __builtin_amdgcn_readfirstlane(tbl.delta[s]);
    f.self = __builtin_amdgcn_readfirstlane(tbl.self[s]);
    const int64_t tok = tbl.tok[s];
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)tok);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)tok >> 32));
    f.tok = (int64_t)(((uint64_t)hi << 32) | lo);
    return f;
}

__device__ __forceinline__ FoundSegment find_segment(const RegSegTable& t, int x, int lane, int) {
    const unsigned long long hit = __ballot(lane < t.n && t.t1 > x);
    const int s = hit ? __builtin_ctzll(hit) : 0;       // x < total: some lane always answers
    FoundSegment f;
    f.seg = s;
    f.first = __builtin_amdgcn_readlane(t.t0, s);
    f.end = __builtin_amdgcn_readlane(t.t1, s);
    f.vis = __builtin_amdgcn_readlane(t.vis, s);
    f.delta = __builtin_amdgcn_readlane(t.delta, s);
    f.self = __builtin_amdgcn_readlane(t.self, s);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)t.tok, s);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)t.tok >> 32), s);
    f.tok = (int64_t)(((uint64_t)hi << 32) | lo);
    return f;
}

// Walks the tiles [next_tile, t_end) of the segment table in order.  All state is wavefront-uniform;
// the segment of the tile handed out last is cached, since most tiles continue their predecessor's.
template <int TILE>
struct TileWalk {
    int next_tile, t_end;
    int c_seg = -1, c_first = 0, c_end = 0, c_vis = 0, c_delta = 0, c_self = 0;
    int64_t c_tok = 0;          // first token of the cached segment in its tensor

    __device__ __forceinline__ TileWalk(int begin, int end) : next_tile(begin), t_end(end) {}

    // The next tile, or a tile with ntok == 0 when none is left.
    template <class Table>
    __device__ __forceinline__ Tile next(const Table& tbl, int lane) {
        Tile d;
        if (next_tile < t_end) {
            if (next_tile >= c_end) {
                const FoundSegment f = find_segment(tbl, next_tile, lane, c_seg);
                c_seg = f.seg;
                c_first = f.first;
                c_end = f.end;
                c_vis = f.vis;
                c_delta = f.delta;
                c_self = f.self;
                c_tok = f.tok;
            }
            d.seg = c_seg;
            d.tok0 = (next_tile - c_first) * TILE;
            d.ntok = max(0, min(TILE, c_vis - d.tok0));
            d.delta = c_delta;
            d.self = c_self;
            ++next_tile;
        } else {
            d.seg = 0; d.tok0 = 0; d.ntok = 0; d.delta = 0; d.self = 0;
        }
        return d;
    }
};

}  // namespace attn

// The kernels that follow the attention kernel of a call (defined with them; `a.dtype` selects the instance).
void launch_combine(const AttnArgs& a, const attn::Plan& p, bool take_pending, hipStream_t s);
bool pending_fit_combine(const AttnArgs& a, const attn::Plan& p);
void launch_mass(const AttnArgs& a, const attn::Plan& p, hipStream_t s);
// S += the masses of the layers whose scores are pending in the ledger (not the current call's): ahead of the fused epilogue
void launch_pending_masses(const AttnArgs& a, const attn::Plan& p, hipStream_t s);
// The fused epilogue keeps every per-document row and the slot partials of a query in LDS: whether they fit.
bool epilogue_fits(const attn::Plan& p, const cf_prune_step* prune);
void launch_epilogue(const AttnArgs& a, const attn::Plan& p, const cf_prune_step* prune, hipStream_t s);
// the same with slot partials in double (the path of cf_attn_plain.hip, which defers nothing)
void launch_mass_f64(const AttnArgs& a, const attn::Plan& p, hipStream_t s);
bool epilogue_fits_f64(const attn::Plan& p, const cf_prune_step* prune);
void launch_epilogue_f64(const AttnArgs& a, const attn::Plan& p, const cf_prune_step* prune, hipStream_t s);

}  // namespace cf
