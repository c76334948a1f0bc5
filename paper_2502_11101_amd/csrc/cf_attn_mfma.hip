// 16-bit MFMA prefill attention for gfx950 (head_dim 128, half-split RoPE pairing).
//
// Work decomposition.  The query rows that share a kv head (all rows of the G = Hq/Hkv heads of
// the group, stacked: row m = g*tq + t) are cut into 16-row blocks; a workgroup owns a run of such blocks of one
// (query, kv head) and a contiguous run of the attended tokens.  Tokens are counted in 32-token tiles that never
// straddle a segment; the tile list of a (query, kv head) is divided evenly over `nsplit` workgroups.  cf_plan.h picks the kernel:
//   * At most 4 row blocks (MHA, short queries: HBM- and latency-bound): attn_tile_kernel, one row block per
//     wavefront, every wavefront loads, stages and computes; two groups of four wavefronts per workgroup stream
//     disjoint runs of tiles.
//   * One row block over a table of at most two entries (decode steps): attn_solo_kernel, every wavefront streams a run of
//     tiles of its own.
//   * More than 4 (GQA groups, long queries): attn_wide_kernel, two or three row
//     blocks per wavefront (up to 192 rows per workgroup), one or two groups of four wavefronts.
// Per tile, in all three:
//   * the tiles ahead (two, or one) are in flight in registers (coalesced 16-byte loads),
//   * the keys are rotated in registers by their segment's relative position shift (Eq. 5; cos/sin per 2-D slice
//     from an fp64-reduced angle) and rounded once to the storage type — rotated keys never return to memory; they
//     go to LDS (attn_solo_kernel: stay in the registers they were loaded to, as matrix operands); V is staged as loaded,
//   * S^T = K Q^T and O^T += V^T P^T run on v_mfma_f32_16x16x32 with the Q fragments resident
//     in registers and the V^T fragments read with transposing LDS reads; the transposed forms keep
//     one query row per lane, so the online softmax (fp32, exp2 domain) needs no cross-lane exchange
//     except when its reference maximum moves.
// Where masses are wanted a wavefront leaves (reference maximum, sum of exp2) per row at the end of each segment.
//
// Where there are several splits a second kernel merges their partial outputs, writes the output rows and reduces the (max, sum) pairs
// over the rows; with one split the attention kernel does.  A last one adds those up to
// per-segment attention mass (the document-wise score of Alg. 2) in a fixed order and adds it to the accumulated scores.  Results cross between the kernels at the
// kernel boundaries: no fences, no atomics on the data path, bit-identical reruns.
#include <type_traits>

#include <hip/hip_ext.h>

#include "cf_attn_tile.h"

namespace cf {
using namespace attn;
namespace {

// ---------------------------------------------------------------------------------------------
// The attention kernel for few stacked rows: the four wavefronts of a group stream the same 32-token
// tiles and own different query rows (wavefront w the 16-row block w), so there is
// nothing to merge inside a group.  Per tile:
//   * every thread's K/V loads for the tile two ahead are in flight in registers (a fixed number of
//     loads per step, so the wait for one tile never covers a later one);
//   * staging: a thread rotates the pairs (c, c + 64) of its 16-byte key chunks (Eq. 5) and writes
//     them [token][channel] to one of two LDS tile buffers; V chunks are copied as loaded, row-major
//     with a 32-byte XOR swizzle; one workgroup barrier per tile;
//   * the tile's math (tile_math).
// Two such groups share a workgroup, stream disjoint runs of tiles and merge at the end.
template <int DT, bool REG_TABLE>
__global__ __launch_bounds__(kThreads * 2, 2) void attn_tile_kernel(AttnArgs a, RopeFreq freq, Plan p) {
    constexpr int kGroups = 2;
    constexpr int kKTile = kTile * kKRow;            // bytes
    constexpr int kVTile = kTile * kD * 2;
    __shared__ SegTable tbl;
    __shared__ __attribute__((aligned(16))) unsigned char k_buf[kGroups][2][kKTile];
    __shared__ __attribute__((aligned(16))) unsigned char v_buf[kGroups][2][kVTile];
    __shared__ __attribute__((aligned(16))) float2 cs_lds[kGroups][2][kHalf];

    const int tid = threadIdx.x & (kThreads - 1);    // thread, wavefront: inside the group of four wavefronts
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int grp = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kThreads);
    const int li = lane & 15, lg = lane >> 4;
    {
        const void *p0 = a.q, *p1 = a.q_off, *p2 = a.q_new_start, *p3 = a.k_store, *p4 = a.v_store, *p5 = a.k_self,
                   *p6 = a.v_self, *p7 = a.segs, *p8 = a.n_seg, *p9 = a.workspace;
        asm volatile("" ::"s"(p0), "s"(p1), "s"(p2), "s"(p3), "s"(p4), "s"(p5), "s"(p6), "s"(p7), "s"(p8), "s"(p9),
                     "s"(a.n_store_tokens), "s"(a.seg_stride), "s"(a.batch), "s"(a.max_tq), "s"(a.n_q_heads),
                     "s"(a.n_kv_heads), "s"(a.scale_log2e), "s"(a.q_stored_start), "s"(p.nsplit), "s"(p.slots),
                     "s"(p.off_massml));
    }

    // grid (split, kv head, query): nothing to divide; one row group (at most four row blocks)
    const int split = blockIdx.x, hkv = blockIdx.y, b = blockIdx.z;
    const int unit = b * a.n_kv_heads + hkv;
    const int group = p.group;
    const QueryHead qh = load_query_head(a, b, REG_TABLE ? lane : (int)threadIdx.x);
    const double my_freq = freq.rev[tid & (kHalf - 1)];
    const int tq = min(qh.tq_raw, a.max_tq);

    // ---- Q fragments first (loads return in order)
    uint4 qf[1][4];
    int trow[1];
    const int row_limit = min(group * tq, p.blocks_rg * 16);
    const bool has_rows = wave * 16 < row_limit;     // wavefront-uniform
    load_q_fragments<1>(a, qh.q0, tq, hkv, group, wave, 0, row_limit, li, lg, qf, trow);

    // at most 64 table entries: every wavefront keeps the table in registers; more: one table in LDS
    RegSegTable rtbl;
    unsigned total;
    if constexpr (REG_TABLE) {
        rtbl = build_reg_table(a, qh, lane, kTile);
        total = (unsigned)rtbl.total;
    } else {
        build_table(a, qh, &tbl, kTile);
        total = (unsigned)tbl.tile0[tbl.n];
    }
    // a group streams a contiguous run of the workgroup's tiles of its own (sub-split `ss`)
    const unsigned nsub = (unsigned)(p.nsplit * kGroups);
    const int ss = split * kGroups + grp;

    // staging items: K (row kr, chunks kj and kj + 8), V (rows vr and vr + 16, chunk vc)
    const int kr = tid >> 3, kj = tid & 7;
    const int vr = tid >> 4, vc = tid & 15;
    struct StageRegs { uint4 ka, kb, v[2]; };
    StageRegs regs0, regs1;

    TileWalk<kTile> walk(split_begin(total, nsub, ss), split_begin(total, nsub, ss + 1));
    // Every call issues the same loads whether or not a tile is left, so the number of loads in flight
    // at any point of the loop is fixed.  Rows past the end of a ragged tile re-read its last row (in
    // bounds; their scores are masked).
    auto fetch = [&](Tile& d, StageRegs& r) {
        if constexpr (REG_TABLE) d = walk.next(rtbl, lane);
        else d = walk.next(tbl, lane);
        const TileSource src = tile_source(a, d, walk.c_tok, hkv);
        const uint32_t k_off = src.last < 0 ? 0u : (uint32_t)min(kr, src.last) * src.row_bytes + 16 * kj;
        r.ka = *reinterpret_cast<const uint4*>(src.k + k_off);
        r.kb = *reinterpret_cast<const uint4*>(src.k + k_off + (src.last < 0 ? 0 : 128));
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const uint32_t off = src.last < 0 ? 0u : (uint32_t)min(vr + 16 * it, src.last) * src.row_bytes + 16 * vc;
            r.v[it] = *reinterpret_cast<const uint4*>(src.v + off);
        }
    };
    Tile d0, d1;
    fetch(d0, regs0);
    fetch(d1, regs1);
    // workgroup-uniform: the longest run among the groups (not needed before the loop, so worked out once the
    // first loads are out)
    int most_tiles = 0;
#pragma unroll
    for (int g = 0; g < kGroups; ++g)
        most_tiles = max(most_tiles, split_begin(total, nsub, split * kGroups + g + 1) - split_begin(total, nsub, split * kGroups + g));

    RowState<1> st;
    st.clear();
    char* ws = static_cast<char*>(a.workspace);
    float2* massml = reinterpret_cast<float2*>(ws + p.off_massml) + (int64_t)unit * p.slots * p.rows_wg;


    // V staging offsets and the transposing reads: lane 16*lg + s addresses row 4*lg + s/4 (+16), 8 bytes at
    // channel 16*db + 4*(s&3)
    const uint32_t vw_off = (uint32_t)vr * 256 + 16 * (vc ^ (2 * (vr & 7)));    // rows vr + 16*it keep (t & 7)
    const int tr_row = 4 * lg + (li >> 2);
    const uint32_t tr_base = (uint32_t)tr_row * 256 + 8 * (li & 3);
    const uint32_t tr_x = (uint32_t)(tr_row & 7) * 32;

    int cs_slot = 0;
    int cur_seg = -1;
    if (d0.ntok > 0 && d0.delta != 0 && tid < kHalf) cs_lds[grp][0][tid] = rope_cos_sin_fast(d0.delta, my_freq);
    __syncthreads();

    // Stage tile `cur` from its registers into buffer `buf`, refill the registers with the tile after
    // `nxt`, prepare the cos/sin table of `nxt`; after the barrier, the math of `cur`.
    auto step = [&](Tile& cur, StageRegs& r, const Tile& nxt, int buf) {
        const Tile cd = cur;
        const bool live = cd.ntok > 0;
        unsigned char* k_lds = k_buf[grp][buf];
        unsigned char* v_lds = v_buf[grp][buf];
        if (live) {
            ChunkAngles ang;
            if (cd.delta != 0) ang = load_chunk_angles(cs_lds[grp][cs_slot] + 8 * kj);
            uint4 ra = r.ka, rb4 = r.kb;
            if (cd.delta != 0) rotate_chunk_pair<DT>(ra, rb4, ang);
            k_tile_write(k_lds, kr, kj, ra);
            k_tile_write(k_lds, kr, kj + 8, rb4);
#pragma unroll
            for (int it = 0; it < 2; ++it) *reinterpret_cast<uint4*>(v_lds + it * 16 * 256 + vw_off) = r.v[it];
        }
        fetch(cur, r);                               // the registers are free again
        if (nxt.ntok > 0 && nxt.seg != cd.seg && nxt.delta != 0) {
            cs_slot ^= 1;
            if (tid < kHalf) cs_lds[grp][cs_slot][tid] = rope_cos_sin_fast(nxt.delta, my_freq);
        }
        __syncthreads();            // tile `cur` is staged; every wavefront is done with the other buffer
        if (!live || !has_rows) return;
        if (cd.seg != cur_seg) {
            if (cur_seg >= 0) emit_segment<1>(st, massml, cur_seg + ss, p.rows_wg, wave, li, lg);
            cur_seg = cd.seg;
#pragma unroll
            for (float& l : st.seg_l) l = 0.f;
        }
        tile_math<DT>(cd, k_lds, v_lds, qf, trow, st, a.scale_log2e, li, lg, tr_base, tr_x);
    };
    // Steps come in pairs and the trip count is the workgroup's: every path round the loop issues the
    // same loads and meets the same barriers.  A group with fewer tiles runs steps without one.
    for (int it = 0; it < most_tiles; it += 2) {
        step(d0, regs0, d1, 0);
        step(d1, regs1, d0, 1);
    }
    if (cur_seg >= 0) emit_segment<1>(st, massml, cur_seg + ss, p.rows_wg, wave, li, lg);

    const StoreArgs ta = store_args(late_args());
    float l_row[1] = {st.l_run[0] + __shfl_xor(st.l_run[0], 16)};       // row sums (each lane holds those of its own tokens so far)
    l_row[0] += __shfl_xor(l_row[0], 32);
    // the second group hands its rows' results (same rows, other tokens) to the first through the tile
    // buffers, which nobody reads any more
    f32x4* red = reinterpret_cast<f32x4*>(&k_buf[0][0][0]);                    // 4 wavefronts x 8 x 64 lanes
    float2* red_ml = reinterpret_cast<float2*>(&v_buf[0][0][0]);               // 4 wavefronts x 16 rows
    __syncthreads();
    if (grp == 1) {
#pragma unroll
        for (int db = 0; db < 8; ++db) red[(wave * 8 + db) * kWave + lane] = st.acc[0][db];
        if (lg == 0) red_ml[wave * 16 + li] = make_float2(st.m_run[0], l_row[0]);
    }
    __syncthreads();
    if (grp == 1 && !ta.slots_here) return;
    float2* const row_ml = red_ml + kWaves * 16;
    if (grp == 0) {
        const float2 o = red_ml[wave * 16 + li];
        const float m = fmaxf(st.m_run[0], o.x);
        const float ms = m == -INFINITY ? 0.f : m;
        const float f0 = __builtin_amdgcn_exp2f(st.m_run[0] - ms), f1 = __builtin_amdgcn_exp2f(o.x - ms);
#pragma unroll
        for (int db = 0; db < 8; ++db) st.acc[0][db] = st.acc[0][db] * f0 + red[(wave * 8 + db) * kWave + lane] * f1;
        l_row[0] = l_row[0] * f0 + o.y * f1;
        st.m_run[0] = m;
        if (ta.slots_here && lg == 0) row_ml[wave * 16 + li] = make_float2(m, wave * 16 + li < row_limit ? l_row[0] : 0.f);
        // a wavefront whose rows are all padding leaves nothing
        if (has_rows) store_partials<DT, 1>(ta, unit, split, wave, st, l_row, lane, qh.q0, tq, hkv, group, 0, row_limit);
    }
    if (!ta.slots_here) return;
    __syncthreads();
    reduce_slots<2 * kWaves>(late_args(), unit, row_ml, (int)threadIdx.x / kWave, lane);
}

// ---------------------------------------------------------------------------------------------
// The attention kernel for one 16-row block over a short table (decode steps: one row per query head of a group) and up to eight splits,
// bound by HBM where there are enough tokens.  With one block attn_tile_kernel has one of four wavefronts do a tile's math while the others wait for it: a
// tile's chain of LDS round trips, ~1 us per 32 KB of a CU.  Here each of a workgroup's eight wavefronts streams tiles of its own
// without a barrier: key fragments straight from memory into the registers the matrix instructions take them from (a lane's 16-byte
// chunks 32 kk + 8 lg of token li hold both channels of each 2-D slice), values through a piece of LDS of the wavefront's own for
// the transposing read.  Two tiles, 256 KB per CU, are in flight.  The eight results meet in LDS at the end.
constexpr int kSoloVRow = 288;                       // bytes per token of a staged V tile
constexpr int kSoloV = kTile * kSoloVRow;

template <int DT>
__global__ __launch_bounds__(kSoloWaves * kWave, 2) void attn_solo_kernel(AttnArgs a, RopeFreq freq, Plan p) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[kSoloWaves * kSoloV];
    __shared__ __attribute__((aligned(16))) float2 cs_lds[kSoloWaves][kHalf];
    __shared__ float2 red_ml[kSoloWaves][16], row_ml[64];
    static_assert(kSoloWaves * kSoloV >= kSoloWaves * 8 * kWave * (int)sizeof(f32x4), "the results reuse the V tiles");

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int li = lane & 15, lg = lane >> 4;
    // grid (split, kv head, query)
    const int split = blockIdx.x, hkv = blockIdx.y, b = blockIdx.z;
    const int unit = b * a.n_kv_heads + hkv;
    const int group = p.group;
    const QueryHead qh = load_query_head(a, b, lane);
    const double my_freq = freq.rev[lane];
    const int tq = min(qh.tq_raw, a.max_tq);
    const int row_limit = group * tq;                // at most 16
    uint4 qf[1][4];
    int trow[1];
    load_q_fragments<1>(a, qh.q0, tq, hkv, group, 0, 0, row_limit, li, lg, qf, trow);
    const RegSegTable rtbl = build_reg_table(a, qh, lane, kTile);
    const unsigned total = (unsigned)rtbl.total;
    // a wavefront's contiguous run of tiles (sub-split `ss`)
    const unsigned nsub = (unsigned)(p.nsplit * kSoloWaves);
    const int ss = split * kSoloWaves + wave;
    TileWalk<kTile> walk(split_begin(total, nsub, ss), split_begin(total, nsub, ss + 1));
    const int my_tiles = walk.t_end - walk.next_tile;

    struct Regs { uint4 k[2][4], v[8]; };            // key fragments [16 tokens][32 channels], V row 4 * i + lane / 16, chunk lane % 16
    auto fetch = [&](Tile& d, Regs& r) {
        d = walk.next(rtbl, lane);
        const TileSource src = tile_source(a, d, walk.c_tok, hkv);
        // rows past a ragged tile's end, and everything where no tile is left, lie past the range and read as zero
        const int range = src.last < 0 ? 0 : src.last * (int)src.row_bytes + 2 * kD;
        const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(src.k), 0, range, 0x00020000);
        const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(src.v), 0, range, 0x00020000);
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            const uint32_t off = (uint32_t)(16 * tb + li) * src.row_bytes + 16 * lg;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                r.k[tb][kk] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rk, off + 64 * kk, 0, 0));
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
            r.v[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rv, (uint32_t)(4 * i + lg) * src.row_bytes + 16 * li, 0, 0));
    };
    Tile d0, d1;
    Regs r0, r1;
    fetch(d0, r0);
    fetch(d1, r1);

    f32x4 acc[8];
#pragma unroll
    for (int db = 0; db < 8; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f, seg_l = 0.f;
    char* ws = static_cast<char*>(a.workspace);
    float2* const massml = reinterpret_cast<float2*>(ws + p.off_massml) + (int64_t)unit * p.slots * p.rows_wg;
    const bool want_mass = a.mass != nullptr;
    int cur_seg = -1;
    // (reference, sum) per row of the segment that ends here
    auto emit = [&]() {
        float tot = seg_l + __shfl_xor(seg_l, 16);
        tot += __shfl_xor(tot, 32);
        if (lg == 0) massml[(int64_t)(cur_seg + ss) * p.rows_wg + li] = make_float2(m_run, tot);
    };
    unsigned char* const v_lds = lds + wave * kSoloV;
    unsigned char* const v_write = v_lds + lg * kSoloVRow + 16 * li;
    const unsigned char* const v_read = v_lds + (4 * lg + (li >> 2)) * kSoloVRow + 8 * (li & 3);
    const float scale_log2e = a.scale_log2e;
    int cs_seg = -1;

    auto step = [&](Tile& d, Regs& r) {
        const Tile cd = d;
        if (cd.seg != cur_seg) {
            if (want_mass && cur_seg >= 0) emit();
            cur_seg = cd.seg;
            seg_l = 0.f;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) *reinterpret_cast<uint4*>(v_write + 4 * i * kSoloVRow) = r.v[i];
        wave_lds_order();                            // what a lane writes here is read by others of the wavefront below
        if (cd.delta != 0) {
            if (cd.seg != cs_seg) {
                cs_seg = cd.seg;
                cs_lds[wave][lane] = rope_cos_sin_fast(cd.delta, my_freq);
            }
            wave_lds_order();
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const ChunkAngles ang = load_chunk_angles(cs_lds[wave] + 32 * kk + 8 * lg);
#pragma unroll
                for (int tb = 0; tb < 2; ++tb) rotate_chunk_pair<DT>(r.k[tb][kk], r.k[tb][kk + 2], ang);
            }
        }
        f32x4 sc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) sc[tb] = Mma<DT>::run(r.k[tb][kk], qf[0][kk], sc[tb]);
        __builtin_amdgcn_sched_barrier(0);
        fetch(d, r);                                 // the registers are free again
        __builtin_amdgcn_sched_barrier(0);
        if (cd.ntok < kTile || cd.self != 0) {
            const int last = (cd.self != 0 ? min(cd.ntok - 1, trow[0] - cd.tok0) : cd.ntok - 1) - 4 * lg;
#pragma unroll
            for (int e = 0; e < 8; ++e) sc[e >> 2][e & 3] = 16 * (e >> 2) + (e & 3) <= last ? sc[e >> 2][e & 3] : -INFINITY;
        }
        // online softmax (exp2 domain) against a stale row maximum (see kProbLimit)
        float pv[8], lsum;
        auto probabilities = [&]() {
            const float m_safe = m_run == -INFINITY ? 0.f : m_run;
            lsum = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                pv[e] = __builtin_amdgcn_exp2f(fmaf(sc[e >> 2][e & 3], scale_log2e, -m_safe));
                lsum += pv[e];
            }
        };
        probabilities();
        if (__any(!(lsum <= kProbLimit) || m_run == -INFINITY)) {
            float mloc = -INFINITY;
#pragma unroll
            for (int e = 0; e < 8; ++e) mloc = fmaxf(mloc, sc[e >> 2][e & 3]);
            mloc *= scale_log2e;                     // scale > 0: max commutes with it
            mloc = fmaxf(mloc, __shfl_xor(mloc, 16));
            mloc = fmaxf(mloc, __shfl_xor(mloc, 32));
            const float m_new = fmaxf(m_run, mloc);
            const float alpha = __builtin_amdgcn_exp2f(m_run - (m_new == -INFINITY ? 0.f : m_new));
            if (__any(alpha != 1.f && m_run != -INFINITY)) {         // nothing accumulated yet: nothing to rescale
#pragma unroll
                for (int db = 0; db < 8; ++db) acc[db] *= alpha;
            }
            l_run *= alpha;
            seg_l *= alpha;
            m_run = m_new;
            probabilities();
        }
        l_run += lsum;
        seg_l += lsum;
        const uint4 pfrag = make_uint4(Mma<DT>::pack(pv[0], pv[1]), Mma<DT>::pack(pv[2], pv[3]), Mma<DT>::pack(pv[4], pv[5]),
                                       Mma<DT>::pack(pv[6], pv[7]));
#pragma unroll
        for (int db = 0; db < 8; ++db) {
            const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)(v_read + 32 * db));
            const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)(v_read + 32 * db + 16 * kSoloVRow));
            const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
            acc[db] = Mma<DT>::run(make_uint4(l2.x, l2.y, h2.x, h2.y), pfrag, acc[db]);
        }
        wave_lds_order();                            // the next step writes over what others read above
    };
    // (left from the middle: with a step skipped the wait for one register set would have to cover the other as well)
    for (int left = my_tiles; left > 0;) {
        step(d0, r0);
        if (--left == 0) break;
        step(d1, r1);
        --left;
    }
    if (want_mass && cur_seg >= 0) emit();

    // ---- the wavefronts' results: wavefront w merges channel block w
    const StoreArgs ta = store_args(late_args());
    float l_row = l_run + __shfl_xor(l_run, 16);
    l_row += __shfl_xor(l_row, 32);
    __syncthreads();                                 // every wavefront is done with its V tile
    f32x4* red = reinterpret_cast<f32x4*>(lds);
#pragma unroll
    for (int db = 0; db < 8; ++db) red[(wave * 8 + db) * kWave + lane] = acc[db];
    if (lg == 0) red_ml[wave][li] = make_float2(m_run, l_row);
    __syncthreads();
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < kSoloWaves; ++w) m = fmaxf(m, red_ml[w][li].x);
    const float ms = m == -INFINITY ? 0.f : m;
    f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
    float l = 0.f;
#pragma unroll
    for (int w = 0; w < kSoloWaves; ++w) {
        const float2 ml = red_ml[w][li];
        const float f = __builtin_amdgcn_exp2f(ml.x - ms);
        l += ml.y * f;
        o += red[(w * 8 + wave) * kWave + lane] * f;
    }
    o *= l > 0.f ? 1.f / l : 0.f;
    const uint2 packed = make_uint2(Mma<DT>::pack(o[0], o[1]), Mma<DT>::pack(o[2], o[3]));
    if (ta.direct_out) {
        if (want_mass) {
            if (wave == 0) row_ml[lane] = make_float2(m, lane < row_limit ? l : 0.f);
            __syncthreads();
            reduce_slots<kSoloWaves>(late_args(), unit, row_ml, wave, lane);
        }
        if (li >= row_limit) return;
        const int gi = (int)div_exact((unsigned)li, (unsigned)tq), t = li - gi * tq;
        uint16_t* op = reinterpret_cast<uint16_t*>(ta.out) + (((int64_t)qh.q0 + t) * ta.n_q_heads + hkv * group + gi) * kD + 16 * wave + 4 * lg;
        *reinterpret_cast<uint2*>(op) = packed;
        return;
    }
    const int64_t part = (int64_t)unit * ta.nsplit + split;
    if (wave == 0 && lg == 0) reinterpret_cast<float2*>(ta.ws + ta.off_ml)[part * ta.rows_wg + li] = make_float2(m, l);
    reinterpret_cast<uint2*>(ta.ws + ta.off_opart)[(part * (ta.rows_wg / 16) * 8 + wave) * kWave + lane] = packed;
}

// ---------------------------------------------------------------------------------------------
// The attention kernel for many stacked rows (GQA groups, long queries), where the instructions that a SIMD can issue are the
// bound: per 32-token tile and 48 rows a wavefront has 48 MFMAs (768 cycles of matrix pipe), about 145 other vector
// instructions and 24 exponentials.  Four wavefronts own NRB 16-row blocks each — 128 or 192 rows of a workgroup, so that a
// staged key serves three row blocks per fragment read — and all of them load, rotate (Eq. 5) and stage the tiles they share.
// A tile passes through two phases of a wavefront:
//   M (matrix)   O^T += V^T P^T of tile t - 1 (8 * NRB MFMAs), S^T = K Q^T of tile t (8 * NRB MFMAs); between the second half of
//                the scores tile t + 1 is rotated in registers and staged; the fragments are read from LDS a few MFMAs ahead of use
//   V (vector)   tile t + 2 requested from memory, softmax of tile t against a stale maximum (kProbLimit)
// The two wavefronts of a SIMD should be in different phases:
//   GROUPS == 2: two groups of four wavefronts stream disjoint runs of the workgroup's tiles, the second group one phase behind the
//                first (a barrier after every phase); their results meet in LDS at the end.  For plans of up to 256 units with ten
//                to thirteen tiles a split and more.
//   GROUPS == 1: one group per workgroup, one barrier per tile.  Past 256 units two workgroups share a CU, and one hides the other's
//                prologue and tail as well: 30 documents of 160 rows and 192 tokens x 32 heads (960 units) 53 us, two groups 77.  Within
//                256 units, where splits are short, a wavefront has its SIMD to itself: the second group's delay and the merge cost more.
// Against the kernel before it (two wavefronts that load and stage, six with two row blocks each, software-pipelined): 64 queries,
// 2 kv heads, 384 rows, 3064 tokens, fp16: 130 -> 111 us (690 TFLOP/s); the 30 documents above 72 -> 53; one query, 4 kv heads, 448
// rows, 7600 tokens 26 us both (more than half of it prologue, merge of the groups and partial store: 13 us + 0.6 per tile).  Two
// tiles in flight instead of one, or the rotation on the matrix cores (diagonal matrices of cosines in three 16-bit parts), no longer
// fit the 256 registers or cost more than they save.
constexpr int kWideK = kTile * kKRow;            // bytes
constexpr int kWideVRow = 288;                       // bytes per token of a staged V tile
constexpr int kWideV = kTile * kWideVRow;

// A register table's fields moved to LDS: the kernel has no registers left to carry them through its loop.
struct LdsSegs {
    const int4* e;              // two per segment: (first token lo, hi, visible, shift), (first tile, end, own block, -)
    int n;
};
__device__ __forceinline__ FoundSegment find_segment(const LdsSegs& t, int x, int, int prev) {
    // the walk goes on from `prev`: the next entry that owns a tile (x < total: there is one)
    int s = prev + 1;
    int4 u = t.e[2 * s], w = t.e[2 * s + 1];
    while (__builtin_amdgcn_readfirstlane(w.y) <= x && s + 1 < t.n) {
        ++s;
        u = t.e[2 * s];
        w = t.e[2 * s + 1];
    }
    FoundSegment f;
    f.seg = s;
    f.tok = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(u.y) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane(u.x));
    f.vis = __builtin_amdgcn_readfirstlane(u.z);
    f.delta = __builtin_amdgcn_readfirstlane(u.w);
    f.first = __builtin_amdgcn_readfirstlane(w.x);
    f.end = __builtin_amdgcn_readfirstlane(w.y);
    f.self = __builtin_amdgcn_readfirstlane(w.z);
    return f;
}

// The lane's index from the hardware: where it is needed seldom, so that nothing derived from it is kept in registers.
__device__ __forceinline__ int lane_anew() {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

// x + the other half's x, for lane pairs 16 and then 32 apart: every lane ends with the sum over the four groups of 16 lanes
__device__ __forceinline__ float add_lane_groups(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// CAUSAL: for calls in one split with several row groups, or whose own block is most of the list (documents encoded offline): half of the
// block's scores are masked.
// The stacked rows are numbered t * group + head, so that a 16-row block sees the own block up to its own last token; a row group ends its
// list there, and a wavefront leaves out the row blocks that see nothing more of it.  Its blocks are every fourth one of the row group (in the
// order of the rows, the missing ones of a group that is not full ahead of all), so that the blocks left out are its first `r0` and the wavefronts
// have equal shares.  The loop exists once for every r0.  So a value that is not finite stays with its tile and the rows behind it; only rows
// ahead of it in a block that sees the tile weigh it by zero.
// Documents encoded and stored, us without and with it (in brackets: row groups in the order of their rows, not the longest lists first): 30 of
// 160 tokens x 32 heads 76.1 and 73.9, 12 of 300 72.1 and 59.8 (67.1); 28 heads over 4, 30 of 160-250 70.6 and 49.8 (56.1), 100 of 100-200 157
// and 120 (128); 12 over 2, 200 of 150-300 215 and 147 (156).  At 160 tokens a workgroup's prologue and the 4 * 39 MB it reads and writes are
// most of its time.
template <int DT, int NRB, int GROUPS, bool REG_TABLE, bool CAUSAL = false>
__global__ __launch_bounds__(kThreads * GROUPS, 2) void attn_wide_kernel(AttnArgs a, RopeFreq freq, Plan p) {
    static_assert(!CAUSAL || (GROUPS == 1 && REG_TABLE), "one split, one group");
    __shared__ SegTable tbl;
    __shared__ double freq_lds[kHalf];
    __shared__ int4 seg_lds[2 * kWave];
    constexpr int kGroupBytes = 2 * kWideK + 3 * kWideV;
    constexpr int kStageBytes = GROUPS * kGroupBytes;
    constexpr int kMergeBytes = GROUPS == 1 ? 0 : 2 * kWaves * NRB * 4 * kWave * (int)sizeof(f32x4);
    __shared__ __attribute__((aligned(16))) unsigned char lds[kStageBytes > kMergeBytes ? kStageBytes : kMergeBytes];
    __shared__ __attribute__((aligned(16))) float2 cs_lds[GROUPS][2][kHalf];
    __shared__ float2 red_ml[GROUPS][kWaves * NRB * 16];

    const int tid = threadIdx.x & (kThreads - 1);
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int grp = GROUPS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / kThreads);
    const int li = lane & 15, lg = lane >> 4;
    unsigned char* const k_lds = lds + grp * kGroupBytes;
    unsigned char* const v_lds = k_lds + 2 * kWideK;

    // grid (split * batch + query, kv head * row groups + row group): a (query, kv head)'s row groups, which read the same keys, come to
    // one XCD where eight divides the first dimension
    const int split = p.nsplit == 1 ? 0 : (int)div_exact(blockIdx.x, (unsigned)a.batch);
    const int b = (int)blockIdx.x - split * a.batch;
    // (CAUSAL: the last row groups, which have the longest lists, first)
    const int by_rg = CAUSAL && p.n_rg > 1 ? (int)div_exact(blockIdx.y, (unsigned)a.n_kv_heads) : 0;
    const int hkv = p.n_rg == 1 ? (int)blockIdx.y : CAUSAL ? (int)blockIdx.y - by_rg * a.n_kv_heads : (int)div_exact(blockIdx.y, (unsigned)p.n_rg);
    const int rg = CAUSAL ? p.n_rg - 1 - by_rg : (int)blockIdx.y - hkv * p.n_rg;
    const int unit = b * p.units_per_b + hkv * p.n_rg + rg;
    const int group = p.group;
    const QueryHead qh = load_query_head(a, b, REG_TABLE ? lane : (int)threadIdx.x);
    if (wave == 0 && grp == 0) freq_lds[lane] = freq.rev[lane];
    const int tq = min(qh.tq_raw, a.max_tq);
    const int row_base = rg * p.blocks_rg * 16;
    const int row_limit = min(group * tq, row_base + p.blocks_rg * 16);
    // the wavefront's block rb: number blk(rb) of the workgroup's, rows row_base + 16 * (blk(rb) - missing) ...
    auto blk = [&](int rb) { return CAUSAL ? rb * kWaves + wave : wave * NRB + rb; };
    const int missing = CAUSAL ? kWaves * NRB - max(0, (row_limit - row_base + 15) / 16) : 0;
    const bool has_rows = CAUSAL ? blk(NRB - 1) >= missing : row_base + wave * NRB * 16 < row_limit;        // wavefront-uniform
    int t_last[NRB];                                 // CAUSAL: the block's last row's place in the own block, -1 without rows
    uint4 qf[NRB][4];
    if constexpr (CAUSAL) {
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
            const int m = row_base + (blk(rb) - missing) * 16 + li;
            const bool valid = blk(rb) >= missing && m < row_limit;
            const int t = valid ? (int)div_exact((unsigned)m, (unsigned)group) : 0, gi = valid ? m - t * group : 0;
            const uint16_t* qp = static_cast<const uint16_t*>(a.q) + (((int64_t)qh.q0 + t) * a.n_q_heads + hkv * group + gi) * kD + 8 * lg;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) qf[rb][kk] = valid ? *reinterpret_cast<const uint4*>(qp + 32 * kk) : make_uint4(0, 0, 0, 0);
            t_last[rb] = __builtin_amdgcn_readfirstlane(
                blk(rb) < missing ? -1 : (int)div_exact((unsigned)min(row_base + (blk(rb) - missing) * 16 + 15, row_limit - 1), (unsigned)group));
        }
    } else {
        int trow[NRB];
        load_q_fragments<NRB>(a, qh.q0, tq, hkv, group, wave * NRB, row_base, row_limit, li, lg, qf, trow);
    }
    RegSegTable rtbl;
    unsigned total;
    if constexpr (REG_TABLE) {
        rtbl = build_reg_table(a, qh, lane, kTile);
        total = (unsigned)rtbl.total;
        if (threadIdx.x < kWave) {
            seg_lds[2 * lane] = make_int4((int)(uint32_t)rtbl.tok, (int)(uint32_t)((uint64_t)rtbl.tok >> 32), rtbl.vis, rtbl.delta);
            seg_lds[2 * lane + 1] = make_int4(rtbl.t0, rtbl.t1, rtbl.self, 0);
        }
    } else {
        build_table(a, qh, &tbl, kTile);
        total = (unsigned)tbl.tile0[tbl.n];
    }
    int own_seg = -1;                                // CAUSAL: the own block, if the list ends with it
    if constexpr (CAUSAL) {
        if (row_limit <= row_base) {
            total = 0;
        } else if (total > 0) {
            const FoundSegment f = find_segment(rtbl, (int)total - 1, lane, -1);
            if (f.self) {
                own_seg = f.seg;
                total = min(total, (unsigned)f.first + div_exact((unsigned)(row_limit - 1), (unsigned)group) / kTile + 1);
            }
        }
    }
    const unsigned nsub = (unsigned)(p.nsplit * GROUPS);
    const int ss = split * GROUPS + grp;

    const int kr = tid >> 3, kj = tid & 7;
    const int vr = tid >> 4, vc = tid & 15;
    struct StageRegs { uint4 ka, kb, v[2]; };
    StageRegs regs;
    // The walk over the sub-split's tiles: next tile, its segment, and where the segment's next tokens start.
    int w_next = split_begin(total, nsub, ss), w_left = 0;
    const int w_end = split_begin(total, nsub, ss + 1);
    Tile w;
    w.seg = -1; w.tok0 = 0; w.ntok = 0; w.delta = 0; w.self = 0;
    int w_slot = 0;                                  // the cos/sin table of its segment
    const char *w_k = static_cast<const char*>(a.workspace), *w_v = w_k;
    uint32_t row_bytes = 0, koff = 0, voff = 0;
    const LdsSegs lsegs{seg_lds, rtbl.n};
    // the next tile's segment, if it starts one, and the segment's cos/sin table
    auto next_segment = [&](auto in_loop) __attribute__((always_inline)) {
        if (w_next >= w_end || w_left > 0) return;
        FoundSegment f;
        if constexpr (!REG_TABLE) f = find_segment(tbl, w_next, lane_anew(), w.seg);
        else if constexpr (decltype(in_loop)::value) f = find_segment(lsegs, w_next, lane_anew(), w.seg);
        else f = find_segment(rtbl, w_next, lane, w.seg);
        w.seg = f.seg;
        w.delta = f.delta;
        w.self = f.self;
        w.tok0 = (w_next - f.first) * kTile;
        w.ntok = 1;
        w_left = f.vis - w.tok0;
        const TileSource src = tile_source(a, w, f.tok, hkv);
        w_k = src.k;
        w_v = src.v;
        if (src.row_bytes != row_bytes) {            // the store's and the own block's rows differ
            row_bytes = src.row_bytes;
            const uint32_t t = (uint32_t)(wave * kWave + lane_anew());
            koff = (t >> 3) * row_bytes + 16 * (t & 7);
            voff = (t >> 4) * row_bytes + 16 * (t & 15);
        }
        if (f.delta != 0) {
            w_slot ^= 1;
            if (wave == 0) {
                const int l = lane_anew();
                cs_lds[grp][w_slot][l] = rope_cos_sin_fast(f.delta, decltype(in_loop)::value ? freq_lds[l] : freq.rev[l]);
            }
        }
    };
    // requests the next tile (d, its table's slot) into r and steps over it
    auto fetch = [&](Tile& d, int& slot, StageRegs& r) __attribute__((always_inline)) {
        d = w;
        d.ntok = w_next < w_end ? min(w_left, kTile) : 0;
        slot = w_slot;
        // rows past a ragged tile's end, and everything where no tile is left, lie past the range and read as zero
        const int range = d.ntok > 0 ? (d.ntok - 1) * (int)row_bytes + 2 * kD : 0;
        const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(w_k), 0, range, 0x00020000);
        const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(w_v), 0, range, 0x00020000);
        r.ka = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rk, koff, 0, 0));
        r.kb = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rk, koff + 128, 0, 0));
        r.v[0] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rv, voff, 0, 0));
        r.v[1] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rv, voff + 16 * row_bytes, 0, 0));
    };
    auto advance = [&]() __attribute__((always_inline)) {
        ++w_next;
        w.tok0 += kTile;
        w_left -= kTile;
        w_k += (int64_t)kTile * row_bytes;
        w_v += (int64_t)kTile * row_bytes;
    };
    unsigned char* const k_write = k_lds + kr * kKRow + 16 * kj;
    unsigned char* const v_write = v_lds + vr * kWideVRow + 16 * vc;
    auto stage = [&](int delta, const StageRegs& r, int slot, int kbuf, int vbuf) __attribute__((always_inline)) {
        uint4 ra = r.ka, rb4 = r.kb;
        rotate_chunk_pair<DT>(ra, rb4, load_chunk_angles(cs_lds[grp][slot] + 8 * kj));
        const bool still = delta == 0;               // bit-exact, and no branch where the matrix instructions run
        ra = make_uint4(still ? r.ka.x : ra.x, still ? r.ka.y : ra.y, still ? r.ka.z : ra.z, still ? r.ka.w : ra.w);
        rb4 = make_uint4(still ? r.kb.x : rb4.x, still ? r.kb.y : rb4.y, still ? r.kb.z : rb4.z, still ? r.kb.w : rb4.w);
        *reinterpret_cast<uint4*>(v_write + vbuf) = r.v[0];
        *reinterpret_cast<uint4*>(v_write + vbuf + 16 * kWideVRow) = r.v[1];
        *reinterpret_cast<uint4*>(k_write + kbuf) = ra;
        *reinterpret_cast<uint4*>(k_write + kbuf + 128) = rb4;
    };

    // The first two tiles are requested together, the first into registers of its own.
    Tile cd, d0;                                     // the tile whose phase M comes next; the tile in `regs` and its table's slot
    int first_slot, slot0;
    StageRegs first;
    next_segment(std::false_type{});
    fetch(cd, first_slot, first);
    advance();
    next_segment(std::false_type{});
    fetch(d0, slot0, regs);
    int most_tiles = 0;
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
        most_tiles = max(most_tiles, split_begin(total, nsub, split * GROUPS + g + 1) - split_begin(total, nsub, split * GROUPS + g));

    RowState<NRB> st;
    st.clear();
    float2* massml = reinterpret_cast<float2*>(static_cast<char*>(a.workspace) + p.off_massml) + (int64_t)unit * p.slots * p.rows_wg;
    const unsigned char* const k_read = k_lds + li * kKRow + 16 * lg;
    const unsigned char* const v_read = v_lds + (4 * lg + (li >> 2)) * kWideVRow + 8 * (li & 3);
    const float scale_log2e = a.scale_log2e;
    int cur_seg = -1;

    short4v vlo[8], vhi[8];                          // V^T fragments of the tile weighed next
    f32x4 sc[NRB][2];                                // its scores
    uint4 pfrag[NRB];                                // its probabilities

    auto read_v = [&](int vbuf, int db0, int db1) __attribute__((always_inline)) {
#pragma unroll
        for (int db = db0; db < db1; ++db) {
            const unsigned char* src = v_read + vbuf + 32 * db;
            vlo[db] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)(src));
            vhi[db] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)(src + 16 * kWideVRow));
        }
    };
    auto weigh = [&](auto first) __attribute__((always_inline)) {
#pragma unroll
        for (int db = 0; db < 8; ++db) {
            const uint2 l2 = __builtin_bit_cast(uint2, vlo[db]), h2v = __builtin_bit_cast(uint2, vhi[db]);
            const uint4 va = make_uint4(l2.x, l2.y, h2v.x, h2v.y);
#pragma unroll
            for (int rb = decltype(first)::value; rb < NRB; ++rb) st.acc[rb][db] = Mma<DT>::run(va, pfrag[rb], st.acc[rb][db]);
        }
    };
    uint4 kf[2][4];
    auto read_k = [&](int kbuf, int kk) __attribute__((always_inline)) {
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) kf[tb][kk] = *reinterpret_cast<const uint4*>(k_read + kbuf + 16 * tb * kKRow + 64 * kk);
    };
    auto scores = [&](auto first, int kk) __attribute__((always_inline)) {
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int rb = decltype(first)::value; rb < NRB; ++rb)
                sc[rb][tb] = Mma<DT>::run(kf[tb][kk], qf[rb][kk], kk == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sc[rb][tb]);
    };
    // phase M, for the blocks from `first` on
    auto matrix_phase = [&](auto first, int vprev, int kcur, int knext, int vnext) __attribute__((always_inline)) {
        constexpr int kBlocks = NRB - decltype(first)::value;
        if constexpr (kBlocks == 0) {
            stage(d0.delta, regs, slot0, knext, vnext);
            advance();
            next_segment(std::true_type{});
            return;
        } else {
        __builtin_amdgcn_sched_barrier(0);
        // channel blocks 0-3 while the V^T fragments of 4-7 come in, those while the first K fragments do
        read_v(vprev, 4, 8);
        weigh(first);
        read_k(kcur, 0);
        read_k(kcur, 1);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
        for (int n = 0; n < 3; ++n) {
            __builtin_amdgcn_sched_group_barrier(0x008, kBlocks, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, kBlocks, 0);
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, kBlocks, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        scores(first, 0);
        scores(first, 1);
        read_k(kcur, 2);
        read_k(kcur, 3);
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            __builtin_amdgcn_sched_group_barrier(0x008, kBlocks, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        // the second half of the scores beside the next tile's rotation
        scores(first, 2);
        scores(first, 3);
        stage(d0.delta, regs, slot0, knext, vnext);
        advance();
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            if (n < 3) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
#pragma unroll
            for (int i = 0; i < kBlocks; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 16 / kBlocks, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        next_segment(std::true_type{});
        }
    };
    auto softmax = [&](auto first, const Tile& cd, int vbuf) __attribute__((always_inline)) {
        constexpr int kFirst = decltype(first)::value;
        if constexpr (kFirst == NRB) return;
        float lsum[NRB];
        auto probabilities = [&](int rb) __attribute__((always_inline)) {
            const float m_safe = st.m_run[rb] == -INFINITY ? 0.f : st.m_run[rb];
            float pv[8];
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                pv[e] = __builtin_amdgcn_exp2f(fmaf(sc[rb][e >> 2][e & 3], scale_log2e, -m_safe));
                s += pv[e];
            }
            lsum[rb] = s;
            pfrag[rb] = make_uint4(Mma<DT>::pack(pv[0], pv[1]), Mma<DT>::pack(pv[2], pv[3]), Mma<DT>::pack(pv[4], pv[5]),
                                   Mma<DT>::pack(pv[6], pv[7]));
        };
        if (cd.ntok < kTile || cd.self != 0) {
            const int l = lane_anew();
            int tqs = CAUSAL ? group : tq;
            asm volatile("" : "+v"(tqs));            // nothing of the division below is kept from tile to tile
#pragma unroll
            for (int rb = kFirst; rb < NRB; ++rb) {
                int lim = cd.ntok;
                if (cd.self != 0) {                  // causal: row m = g * tq + t (CAUSAL: t * group + g) sees the own block up to its t
                    const int m = row_base + (blk(rb) - missing) * 16 + (l & 15);
                    const int t = CAUSAL ? (int)div_exact((unsigned)max(m, 0), (unsigned)tqs) : m - (int)div_exact((unsigned)m, (unsigned)tqs) * tqs;
                    lim = min(lim, t - cd.tok0 + 1);
                }
                lim -= 4 * (l >> 4);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    sc[rb][e >> 2][e & 3] = 16 * (e >> 2) + (e & 3) < lim ? sc[rb][e >> 2][e & 3] : -INFINITY;
            }
        }
#pragma unroll
        for (int rb = kFirst; rb < NRB; ++rb) probabilities(rb);
        bool any_off = false;
#pragma unroll
        for (int rb = kFirst; rb < NRB; ++rb) any_off = any_off || !(lsum[rb] <= kProbLimit) || st.m_run[rb] == -INFINITY;
        if (__any(any_off)) {
#pragma unroll
            for (int rb = kFirst; rb < NRB; ++rb) {
                float mloc = -INFINITY;
#pragma unroll
                for (int e = 0; e < 8; ++e) mloc = fmaxf(mloc, sc[rb][e >> 2][e & 3]);
                mloc *= scale_log2e;
                mloc = fmaxf(mloc, __shfl_xor(mloc, 16));
                mloc = fmaxf(mloc, __shfl_xor(mloc, 32));
                const float m_old = st.m_run[rb];
                const float m_new = fmaxf(m_old, mloc);
                const float alpha = __builtin_amdgcn_exp2f(m_old - (m_new == -INFINITY ? 0.f : m_new));
                st.l_run[rb] *= alpha;
                st.seg_l[rb] *= alpha;
                st.m_run[rb] = m_new;
#pragma unroll
                for (int db = 0; db < 8; ++db) st.acc[rb][db] *= alpha;
                probabilities(rb);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        read_v(vbuf, 0, 4);
#pragma unroll
        for (int rb = kFirst; rb < NRB; ++rb) {
            st.seg_l[rb] += lsum[rb];
        }
    };
    // (reference, segment sum) per row for the segment's slot
    auto emit = [&](int seg) __attribute__((always_inline)) {
        float tot[NRB];
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) tot[rb] = add_lane_groups(st.seg_l[rb]);
        const int l = lane_anew();
        if (l < 16) {
            float2* dst = massml + (int64_t)(seg + ss) * p.rows_wg + blk(0) * 16 + l;
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) dst[16 * (blk(rb) - blk(0))] = make_float2(st.m_run[rb], tot[rb]);
        }
    };
    // phase V, for the blocks from `first` on
    auto vector_phase = [&](auto first, const Tile& cd, int vbuf) __attribute__((always_inline)) {
        if (cd.ntok <= 0) {
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) pfrag[rb] = make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int db = 0; db < 4; ++db) vlo[db] = vhi[db] = short4v{0, 0, 0, 0};      // (an infinity times zero)
            return;
        }
        if (cd.seg != cur_seg) {
            if (cur_seg >= 0) emit(cur_seg);
            cur_seg = cd.seg;
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) { st.l_run[rb] += st.seg_l[rb]; st.seg_l[rb] = 0.f; }
        }
        softmax(first, cd, vbuf);
    };
    // the first of the wavefront's blocks that sees anything of a tile (all after it do); it only grows along the list
    auto first_block = [&](const Tile& d) __attribute__((always_inline)) {
        int r0 = 0;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) r0 += t_last[rb] < (d.seg == own_seg ? d.tok0 : 0) ? 1 : 0;
        return r0;
    };
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) pfrag[rb] = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int db = 0; db < 8; ++db) vlo[db] = vhi[db] = short4v{0, 0, 0, 0};

    // (the first phase weighs nothing, with probabilities of zero: what it reads of the buffer before must be finite)
    *reinterpret_cast<uint4*>(v_write + 2 * kWideV) = make_uint4(0, 0, 0, 0);
    *reinterpret_cast<uint4*>(v_write + 2 * kWideV + 16 * kWideVRow) = make_uint4(0, 0, 0, 0);
    __syncthreads();                                 // the cos/sin tables of the first two tiles, the segment table in LDS
    stage(cd.delta, first, first_slot, 0, 0);
    __syncthreads();                                 // tile 0 is staged
    if (GROUPS == 2 && grp == 1) __syncthreads();    // the second group runs one phase behind
    // step t: d0 / regs hold tile t + 1, after it tile t + 2
    int kcur = 0, vprev = 2 * kWideV, vcur = 0, vnext = kWideV;
    int it = 0, r_prev = CAUSAL ? first_block(cd) : 0;       // the first block of the tile before
    auto steps = [&](auto first) __attribute__((always_inline)) {
        constexpr int kFirst = decltype(first)::value;       // (the probabilities of the blocks before it are zero since their last tile)
        for (; it < most_tiles && (!CAUSAL || r_prev <= kFirst); ++it) {
            __builtin_amdgcn_s_setprio(1);
            matrix_phase(first, vprev, kcur, kWideK - kcur, vnext);
            __builtin_amdgcn_s_setprio(0);
            if (GROUPS == 2) __syncthreads();
            const Tile cur = cd;
            cd = d0;
            fetch(d0, slot0, regs);
            vector_phase(first, cur, vcur);
            if constexpr (CAUSAL) r_prev = first_block(cur);
            kcur = kWideK - kcur;
            const int v = vprev;
            vprev = vcur;
            vcur = vnext;
            vnext = v;
            __syncthreads();
        }
    };
    steps(std::integral_constant<int, 0>{});
    if constexpr (CAUSAL) {
        steps(std::integral_constant<int, 1>{});
        steps(std::integral_constant<int, 2>{});
        if constexpr (NRB == 3) steps(std::integral_constant<int, 3>{});
    }
    if (GROUPS == 2 && grp == 0) __syncthreads();
    // (CAUSAL: the last tile for the blocks that see any of it, not times zero for the others: it may hold an infinity)
    auto close = [&](auto first) __attribute__((always_inline)) { read_v(vprev, 4, 8); weigh(first); };
    if (!CAUSAL || r_prev == 0) close(std::integral_constant<int, 0>{});
    else if (r_prev == 1) close(std::integral_constant<int, 1>{});
    else if (NRB == 3 && r_prev == 2) close(std::integral_constant<int, 2>{});
    if (has_rows && cur_seg >= 0) emit(cur_seg);

    const StoreArgs ta = store_args(late_args());
    const int lane_t = lane_anew(), li_t = lane_t & 15, lg_t = lane_t >> 4;      // (not kept through the loop)
    float l_row[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
        st.l_run[rb] += st.seg_l[rb];
        l_row[rb] = st.l_run[rb] + __shfl_xor(st.l_run[rb], 16);
        l_row[rb] += __shfl_xor(l_row[rb], 32);
    }
    if (GROUPS == 1) {
        if (ta.slots_here && lg_t == 0) {
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) {
                const int row = blk(rb) * 16 + li_t;
                red_ml[0][row] = make_float2(st.m_run[rb], blk(rb) >= missing && row_base + row - 16 * missing < row_limit ? l_row[rb] : 0.f);
            }
        }
        if constexpr (CAUSAL) {
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) {
                if (blk(rb) < missing) continue;
                const int m = row_base + (blk(rb) - missing) * 16 + li_t, mc = min(m, row_limit - 1);      // (every lane takes part in the exchange)
                const int t = (int)div_exact((unsigned)mc, (unsigned)group), gi = mc - t * group;
                const float inv = l_row[rb] > 0.f ? 1.f / l_row[rb] : 0.f;
                uint16_t* op = reinterpret_cast<uint16_t*>(ta.out) + (((int64_t)qh.q0 + t) * ta.n_q_heads + hkv * group + gi) * kD;
#pragma unroll
                for (int db = 0; db < 8; db += 2) store_row_pair<DT>(op, db, st.acc[rb][db] * inv, st.acc[rb][db + 1] * inv, lg_t, m < row_limit);
            }
        } else if (has_rows) store_partials<DT, NRB>(ta, unit, split, wave * NRB, st, l_row, lane_t, qh.q0, tq, hkv, group, row_base, row_limit);
        if (!ta.slots_here) return;
        __syncthreads();
        reduce_slots<kWaves>(late_args(), unit, red_ml[0], wave, lane_t);
        return;
    }
    __syncthreads();
    f32x4* red = reinterpret_cast<f32x4*>(lds);
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
        if (lg_t == 0) red_ml[grp][(wave * NRB + rb) * 16 + li_t] = make_float2(st.m_run[rb], l_row[rb]);
        // the first group keeps channel blocks 0-3, the second 4-7
        f32x4* dst = red + (((grp * kWaves + wave) * NRB + rb) * 4) * kWave + lane_t;
        if (grp == 0) {
#pragma unroll
            for (int db = 0; db < 4; ++db) dst[db * kWave] = st.acc[rb][4 + db];
        } else {
#pragma unroll
            for (int db = 0; db < 4; ++db) dst[db * kWave] = st.acc[rb][db];
#pragma unroll
            for (int db = 0; db < 4; ++db) st.acc[rb][db] = st.acc[rb][4 + db];
        }
    }
    __syncthreads();
    if (!has_rows && !ta.slots_here) return;
    const int64_t part = (int64_t)unit * ta.nsplit + split;
    float2* const row_ml = reinterpret_cast<float2*>(&cs_lds[0][0][0]);          // nobody reads the angles any more
    static_assert(sizeof(cs_lds) >= kWaves * NRB * 16 * sizeof(float2) || GROUPS == 1, "room for the rows");
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
        if (!has_rows) continue;
        const float2 o = red_ml[grp ^ 1][(wave * NRB + rb) * 16 + li_t];
        const float m = fmaxf(st.m_run[rb], o.x);
        const float ms = m == -INFINITY ? 0.f : m;
        const float f0 = __builtin_amdgcn_exp2f(st.m_run[rb] - ms), f1 = __builtin_amdgcn_exp2f(o.x - ms);
        const f32x4* src = red + ((((grp ^ 1) * kWaves + wave) * NRB + rb) * 4) * kWave + lane_t;
        // the sums in the groups' order, so that both come to the same row sum
        const float l = grp == 0 ? l_row[rb] * f0 + o.y * f1 : o.y * f1 + l_row[rb] * f0;
        const float inv = l > 0.f ? 1.f / l : 0.f;
        const int blk = wave * NRB + rb;
        f32x4 o4[4];
#pragma unroll
        for (int db = 0; db < 4; ++db) o4[db] = (st.acc[rb][db] * f0 + src[db * kWave] * f1) * inv;
        if (ta.direct_out) {
            const int row = row_base + blk * 16 + li_t, mrow = min(row, row_limit - 1);
            if (ta.slots_here && grp == 0 && lg_t == 0) row_ml[blk * 16 + li_t] = make_float2(m, row < row_limit ? l : 0.f);
            const int gi = (int)div_exact((unsigned)mrow, (unsigned)tq), t = mrow - gi * tq;
            uint16_t* op = reinterpret_cast<uint16_t*>(ta.out) + (((int64_t)qh.q0 + t) * ta.n_q_heads + hkv * group + gi) * kD + 64 * grp;
#pragma unroll
            for (int db = 0; db < 4; db += 2) store_row_pair<DT>(op, db, o4[db], o4[db + 1], lg_t, row < row_limit);
        } else {
            float2* ml = reinterpret_cast<float2*>(ta.ws + ta.off_ml) + part * ta.rows_wg;
            if (grp == 0 && lg_t == 0) ml[blk * 16 + li_t] = make_float2(m, l);
            uint2* opart = reinterpret_cast<uint2*>(ta.ws + ta.off_opart) + ((part * ta.rows_wg / 16 + blk) * 8 + 4 * grp) * kWave + lane_t;
#pragma unroll
            for (int db = 0; db < 4; ++db) opart[db * kWave] = make_uint2(Mma<DT>::pack(o4[db][0], o4[db][1]), Mma<DT>::pack(o4[db][2], o4[db][3]));
        }
    }
    if (!ta.slots_here) return;
    if (!has_rows && grp == 0 && lg_t == 0) {
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) row_ml[(wave * NRB + rb) * 16 + li_t] = make_float2(0.f, 0.f);
    }
    __syncthreads();
    reduce_slots<2 * kWaves>(late_args(), unit, row_ml, (int)threadIdx.x / kWave, lane_t);
}

}  // namespace

bool mfma_path_supported(const cf_layer_desc* d) {
    return (d->dtype == CF_BF16 || d->dtype == CF_F16) && d->head_dim == kD && d->rope_pairing == CF_ROPE_HALF;
}

static bool mfma_shape_ok(int seg_stride) { return seg_stride <= kMaxSegs; }

size_t mfma_workspace_bytes(const cf_layer_desc* d, int32_t batch, int32_t max_tq, int32_t seg_stride,
                            int64_t max_kv_tokens) {
    if (!mfma_shape_ok(seg_stride)) return generic_workspace_bytes(d, batch, max_tq, seg_stride);
    return workspace_bytes(d->n_q_heads, d->n_kv_heads, batch, max_tq, seg_stride, max_kv_tokens);
}

size_t mfma_call_bytes(const cf_layer_desc* d, int32_t batch, int32_t max_tq, int32_t seg_stride, int64_t max_kv_tokens, size_t given) {
    if (!mfma_shape_ok(seg_stride)) return generic_workspace_bytes(d, batch, max_tq, seg_stride);
    return make_plan(d->n_q_heads, d->n_kv_heads, batch, max_tq, seg_stride, max_kv_tokens, given).total;
}

cf_status launch_attention_mfma(const AttnArgs& a, const RopeFreq& f, hipStream_t s, const cf_prune_step* prune) {
    if (!mfma_shape_ok(a.seg_stride)) {
        cf_status st = launch_attention_generic(a, f, s);
        return st != CF_OK || !prune ? st : launch_prune_step(a, prune, s);
    }
    const Plan p = make_plan(a.n_q_heads, a.n_kv_heads, a.batch, a.max_tq, a.seg_stride, a.max_kv_tokens, a.workspace_bytes);
    const dim3 grid3((unsigned)p.nsplit, (unsigned)a.n_kv_heads, (unsigned)a.batch);     // attn_tile_kernel's and attn_solo_kernel's
    const dim3 grid2((unsigned)(p.nsplit * a.batch), (unsigned)p.units_per_b);           // attn_wide_kernel's
    if (a.batch > 65535 || !wide_grid_ok(a.n_kv_heads, p)) {
        set_error("neither batch nor n_kv_heads * row groups may exceed 65535 on this path");
        return CF_ERR_UNSUPPORTED;
    }
    const bool reg_table = a.seg_stride <= kRegEntries;      // the attention kernels keep a table this small in registers
    // the attention kernel's launch carries the profiling aid's start/stop events (null when it is off)
    hipEvent_t ev_start = nullptr, ev_stop = nullptr;
    profile_kernel_pair(&ev_start, &ev_stop);
#define CF_LAUNCH_TIMED(KERNEL, GRID, BLOCK)                                                          \
    do {                                                                                              \
        static_assert(std::is_same_v<decltype(&KERNEL), LateArgsKernel>);                             \
        if (ev_start) hipExtLaunchKernelGGL(KERNEL, GRID, BLOCK, 0, s, ev_start, ev_stop, 0, a, f, p); \
        else hipLaunchKernelGGL(KERNEL, GRID, BLOCK, 0, s, a, f, p);                                  \
    } while (0)
#define CF_LAUNCH_WIDE(DT, GROUPS)                                                                                            \
    if (p.nrb == 2) {                                                                                                         \
        if (reg_table) CF_LAUNCH_TIMED((attn_wide_kernel<DT, 2, GROUPS, true>), grid2, dim3(GROUPS * kThreads));              \
        else CF_LAUNCH_TIMED((attn_wide_kernel<DT, 2, GROUPS, false>), grid2, dim3(GROUPS * kThreads));                       \
    } else {                                                                                                                  \
        if (reg_table) CF_LAUNCH_TIMED((attn_wide_kernel<DT, 3, GROUPS, true>), grid2, dim3(GROUPS * kThreads));              \
        else CF_LAUNCH_TIMED((attn_wide_kernel<DT, 3, GROUPS, false>), grid2, dim3(GROUPS * kThreads));                       \
    }
#define CF_LAUNCH_DT(DT)                                                                                                       \
    if (p.groups == kSoloWaves) {                                                                                                             \
        CF_LAUNCH_TIMED((attn_solo_kernel<DT>), grid3, dim3(kSoloWaves * kWave));                                              \
    } else if (!p.wide) {                                                                                                      \
        if (reg_table) CF_LAUNCH_TIMED((attn_tile_kernel<DT, true>), grid3, dim3(2 * kThreads));                            \
        else CF_LAUNCH_TIMED((attn_tile_kernel<DT, false>), grid3, dim3(2 * kThreads));                                     \
    } else {                                                                                                                   \
        if (p.wide == 2) {                                                                                                     \
            if (p.nrb == 2) CF_LAUNCH_TIMED((attn_wide_kernel<DT, 2, 1, true, true>), grid2, dim3(kThreads));                   \
            else CF_LAUNCH_TIMED((attn_wide_kernel<DT, 3, 1, true, true>), grid2, dim3(kThreads));                              \
        } else if (p.groups == 2) { CF_LAUNCH_WIDE(DT, 2) } else { CF_LAUNCH_WIDE(DT, 1) }                                             \
    }                                                                                                                          \
    CF_HIP(hipGetLastError());
    if (a.dtype == CF_BF16) { CF_LAUNCH_DT(CF_BF16) } else { CF_LAUNCH_DT(CF_F16) }
#undef CF_LAUNCH_DT
#undef CF_LAUNCH_WIDE
#undef CF_LAUNCH_TIMED
    const bool combine = !p.direct_out;              // one split: the attention kernel has written the rows and reduced the slots
    // before a fused epilogue the pending score parts are taken in by one more row of the combine kernel's grid
    const bool pending_beside = combine && !a.defer && prune && a.n_pending > 0 && epilogue_fits(p, prune) && pending_fit_combine(a, p);
    if (combine) launch_combine(a, p, pending_beside, s);
    CF_HIP(hipGetLastError());
    if (a.defer) return CF_OK;                       // the slot partials stay in the ledger for a later call
    if (prune) {
        if (epilogue_fits(p, prune)) {
            if (a.n_pending > 0 && !pending_beside) launch_pending_masses(a, p, s);
            launch_epilogue(a, p, prune, s);
        } else {
            launch_mass(a, p, s);
            CF_HIP(hipGetLastError());
            return launch_prune_step(a, prune, s);
        }
    } else if (a.mass != nullptr) {
        launch_mass(a, p, s);
    }
    CF_HIP(hipGetLastError());
    return CF_OK;
}

}  // namespace cf
