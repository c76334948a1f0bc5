// What follows the attention kernel of a call on the 16-bit path: the merge of the splits' partial outputs
// (with the slot partial masses as a by-product), the per-segment mass reduction, and the fused layer epilogue
// (masses, S += mass, ranking, allocation, next segment table).
#include <type_traits>

#include "cf_attn_plan.h"

namespace cf {
using namespace attn;
namespace {

__device__ __forceinline__ void pending_masses_block(const AttnArgs& a, const Plan& p, int b, int n_parts, int write_mass,
                                                     float (*m_all)[kWave]);

// Second kernel, where there are several splits: merges the splits' partial outputs, writes the output rows and, with MASS, reduces every
// (segment, split) slot's (max, sum) pairs over a pass's 64 rows to sum * exp2(max - row max) / row sum, which the mass kernel then only
// has to add up.  A wavefront owns one (16-row block, 16 channels) of a unit = (query, kv head, row group); the wavefronts of a (unit, pass)
// share its slots.  At these sizes it is bound by its two dependent round trips (arguments, then one batch of loads), so a wavefront works
// out the statistics of its rows for itself, from loads of that batch, and there is neither LDS nor a barrier behind them.  With the statistics
// shared through LDS by a workgroup and three barriers: 32 units x 7 splits x 1 row 4.2 -> 3.3 us (the decode step 11.5 -> 10.6), 32 x 8 x 48
// rows 4.2 -> 3.5 (32 such layers 674 -> 643), 16 x 16 x 112 rows 6.2 -> 4.9, 128 x 2 x 7 rows 5.6 -> 4.7.
// NS: splits whose statistics are held in registers.  spread: log2 of the channel blocks of a workgroup (0 for more than two row blocks,
// 1 for two, 2 for one, as in a decode step), so that no wavefront is left without rows.
// With take_pending the grid has one more row of workgroups, the first: its first workgroup, per query, takes the ledger's pending
// score parts in beside the merge (pending_masses_block), which takes longer than a merge, the others leave at once.
template <int DT, int NS, bool MASS>
__global__ __launch_bounds__(kThreads) void attn_combine_kernel(AttnArgs a, Plan p, int take_pending, int spread) {
    if constexpr (MASS) {
        __shared__ float m_all[kMaxPending + 1][kWave];
        if (take_pending && blockIdx.y == 0) {
            if (blockIdx.x == 0) pending_masses_block(a, p, __builtin_amdgcn_readfirstlane(blockIdx.z), a.n_pending, 0, m_all);
            return;
        }
    }
    constexpr int kPre = 8;                      // splits whose partial outputs are fetched before the statistics are ready
    constexpr int kSv = 8;                       // slot statistics fetched up front per wavefront

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int li = lane & 15, lg = lane >> 4;
    char* ws = static_cast<char*>(a.workspace);
    // grid (kv head * row groups + row group, channel blocks + their number * pass, query): where eight divides the first dimension a unit's
    // workgroups come to one XCD, which reads its statistics once and puts its output lines together (16 units 7.3 -> 6.6 us, 32 units 4.4 -> 4.3 before the above)
    const int y = (int)blockIdx.y - (MASS ? take_pending : 0);
    const int blk_in = wave & (kWaves - 1) >> spread;                              // row block inside the pass
    const int dbq = (y & 7 >> spread) << spread | wave >> (2 - spread), pass = y >> (3 - spread);
    const int b = blockIdx.z;
    const int hkv = p.n_rg == 1 ? (int)blockIdx.x : (int)div_exact(blockIdx.x, (unsigned)p.n_rg);
    const int rg = (int)blockIdx.x - hkv * p.n_rg;
    const int unit = b * p.units_per_b + (int)blockIdx.x;
    const int q0 = a.q_off[b], q1 = a.q_off[b + 1];
    // with MASS lane r holds row r of the pass, which the slots are reduced over, else the row of the lane's partial outputs
    const int row = MASS ? lane : blk_in * 16 + li;
    const float2* ml = reinterpret_cast<const float2*>(ws + p.off_ml) + (int64_t)unit * p.nsplit * p.rows_wg + pass * 64 + row;
    const uint2* opart = reinterpret_cast<const uint2*>(ws + p.off_opart) + (int64_t)unit * p.nsplit * p.rows_wg * (kD / 4);
    const uint2* src = opart + ((int64_t)(pass * kWaves + blk_in) * 8 + dbq) * kWave + lane;
    auto widen = [](uint2 w) { return f32x4{Mma<DT>::lo(w.x), Mma<DT>::hi(w.x), Mma<DT>::lo(w.y), Mma<DT>::hi(w.y)}; };
    const int64_t split_stride = (int64_t)p.rows_wg / 16 * 8 * kWave;
    const float2* massml = reinterpret_cast<const float2*>(ws + p.off_massml) + (int64_t)unit * p.slots * p.rows_wg + pass * 64 + lane;
    const int k_first = dbq * (kWaves >> spread) + blk_in, k_step = 8 * kWaves >> spread;

    // Everything this wavefront reads is requested up front — row statistics, partial outputs of the first splits,
    // the first slot statistics — so the round trips to memory overlap.  Every load is unconditional (a clamped,
    // in-bounds address; what lies past the end is dropped afterwards): a load inside a branch makes the compiler
    // wait for it before the branch ends, which would put the round trips one behind the other.
    // (A wavefront whose 16 rows are all padding reads what an earlier call left there: never stored; not waiting for
    // the query's length here saves a round trip.)
    float2 st[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) st[s] = ml[(int64_t)min(s, p.nsplit - 1) * p.rows_wg];
    uint2 pre[kPre];
#pragma unroll
    for (int s = 0; s < kPre; ++s) pre[s] = src[min(s, p.nsplit - 1) * split_stride];
    float2 sv[kSv];
    if constexpr (MASS) {
#pragma unroll
        for (int j = 0; j < kSv; ++j) sv[j] = massml[(int64_t)min(k_first + j * k_step, p.slots - 1) * p.rows_wg];
    }
    __builtin_amdgcn_sched_barrier(0);
    const int tq = min(q1 - q0, a.max_tq);
    const int n_rows = p.group * tq;
    const int row_base = rg * p.blocks_rg * 16;
    const int rows_here = min(p.blocks_rg * 16, n_rows - row_base);
    // A row's maximum, and its sum in four interleaved parts; a split's weight stays unnormalised (its rows arrive divided by their own
    // sum), the rows are divided by their sum once at the end.
    float m = -INFINITY;
#pragma unroll
    for (int s = 0; s < NS; ++s) m = fmaxf(m, st[s].x);
    m = m == -INFINITY ? 0.f : m;
    float z4[4] = {0.f, 0.f, 0.f, 0.f}, weight[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        weight[s] = s < p.nsplit ? st[s].y * exp2f(st[s].x - m) : 0.f;
        z4[s & 3] += weight[s];
    }
    const float z = ((z4[0] + z4[1]) + z4[2]) + z4[3];
    const float inv = z > 0.f ? 1.f / z : 0.f;
    auto of_block = [&](float x) { return MASS ? __shfl(x, blk_in * 16 + li) : x; };
    f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s0 = 0; s0 < NS; s0 += kPre) {
        if (s0 >= p.nsplit) break;
        if (s0 > 0) {                                // further splits, eight loads at a time (unconditional, as above)
#pragma unroll
            for (int i = 0; i < kPre; ++i) pre[i] = src[min(s0 + i, p.nsplit - 1) * split_stride];
        }
        float w[kPre];
#pragma unroll
        for (int i = 0; i < kPre; ++i) w[i] = of_block(weight[s0 + i]);
#pragma unroll
        for (int i = 0; i < kPre; ++i)
            if (s0 + i < p.nsplit) o += widen(pre[i]) * w[i];
    }
    o *= of_block(inv);
    const int lrow = pass * 64 + blk_in * 16 + li;
    if (lrow < rows_here) {
        const int m2 = row_base + lrow;
        const int gi = (int)div_exact((unsigned)m2, (unsigned)tq), t = m2 - gi * tq;
        uint16_t* op = static_cast<uint16_t*>(a.out) + (((int64_t)q0 + t) * a.n_q_heads + hkv * p.group + gi) * kD + 16 * dbq + 4 * lg;
        uint2 pk;
        pk.x = Mma<DT>::pack(o[0], o[1]);
        pk.y = Mma<DT>::pack(o[2], o[3]);
        *reinterpret_cast<uint2*>(op) = pk;
    }
    // slot partials: slot k = segment + split; slots no split wrote this call hold stale pairs and
    // give meaningless numbers that the mass kernel never reads
    if constexpr (MASS) {
        float* masspart = reinterpret_cast<float*>(ws + p.off_masspart + (size_t)a.n_pending * p.masspart_bytes) + ((int64_t)unit * p.nrb + pass) * p.slots;
        const float2 stat = make_float2(m, pass * 64 + lane < rows_here ? inv : 0.f);   // padding rows carry no mass
        auto reduce = [&](int k, float2 v) {
            const float c = wave_sum_dpp(stat.y > 0.f ? v.y * exp2f(v.x - stat.x) * stat.y : 0.f);
            if (lane == 0 && k < p.slots) masspart[k] = c;
        };
#pragma unroll
        for (int j = 0; j < kSv; ++j)
            if (k_first + j * k_step < p.slots) reduce(k_first + j * k_step, sv[j]);
        for (int k = k_first + kSv * k_step; k < p.slots; k += k_step) reduce(k, massml[(int64_t)k * p.rows_wg]);
    }
}

// Per-segment attention mass of one query, by the whole workgroup, in a fixed order: first every
// slot's partials are added over the (unit, pass) parts, then a segment adds the slots of the
// splits that hold its tiles.  A split between a segment's first and last may own no tile at
// all (fewer tiles than splits): its slot was not written by this call and is skipped.
// `parts`: [nparts][slots] floats, in LDS (stage == nullptr; overwritten) or in memory (stage: kMassStage floats
// of LDS).  `on_mass(s, m)` is called once per segment.  Both forms add in the same order: the parts of a
// column in groups of eight, each group from zero, then the group sums from zero.
// Sum of n <= 8 values `pitch` floats apart, added in order from zero.  A full group's loads all go out
// before the first add (a loop with a run-time bound would wait for each in turn).
template <class T>
__device__ __forceinline__ T group_sum(const T* x, int pitch, int n) {
    T gs = 0;
    if (n == 8) {
        T v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = x[i * pitch];
#pragma unroll
        for (int i = 0; i < 8; ++i) gs += v[i];
    } else {
        for (int i = 0; i < n; ++i) gs += x[i * pitch];
    }
    return gs;
}

template <class T>
struct MassScratch {
    T colsum[kMaxSegs + kMaxSub];
    int32_t sub_begin[kMaxSub + 1];
    float seg_mass[kMaxSegs];               // every entry's mass, for the per-document sums
};

// S += s^l (Alg. 2) without atomics, so that the sum does not depend on timing when a document slot is fed by
// several table entries: the first entry of a slot adds up the masses of all entries of that slot in table
// order and is the only one that touches the slot's score.
// Block form: `doc` and `seg_mass` of the n entries in LDS; `score` has `stride` slots (LDS or memory).
__device__ __forceinline__ void add_doc_scores_block(const int32_t* doc, const float* seg_mass, int n, float* score, int stride) {
    for (int s = threadIdx.x; s < n; s += blockDim.x) {
        const int d = doc[s];
        if (d < 0 || d >= stride) continue;
        bool first = true;
        float sum = seg_mass[s];
        for (int j = 0; j < n; ++j) {
            if (doc[j] != d) continue;
            if (j < s) first = false;
            else if (j > s) sum += seg_mass[j];
        }
        if (first) score[d] += sum;
    }
}
// Bitwise OR over the 64 lanes of a wavefront, handed to every lane (DPP row shifts, then the two row broadcasts).
__device__ __forceinline__ uint32_t wave_or_u32(uint32_t x) {
    int v = (int)x;
    v |= __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v |= __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v |= __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v |= __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v |= __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    v |= __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return (uint32_t)__builtin_amdgcn_readlane(v, 63);
}
// Wavefront form: lane s < n holds entry s's slot (doc) and mass.  With at most 64 document slots a bit mask tells whether
// every slot is fed by one entry only — the usual table — and then every entry adds its own mass (the same single
// addend as below); otherwise the loop runs once per table entry.
__device__ __forceinline__ bool one_entry_per_slot(int doc, int n, int lane, int stride) {
    if (stride > kWave) return false;
    const bool valid = lane < n && doc >= 0 && doc < stride;
    const unsigned long long bit = valid ? 1ull << doc : 0ull;
    const int slots_fed = __builtin_popcount(wave_or_u32((uint32_t)bit)) + __builtin_popcount(wave_or_u32((uint32_t)(bit >> 32)));
    return slots_fed == __builtin_popcountll(__ballot(valid));
}
__device__ __forceinline__ void add_doc_scores_wave(int doc, float m, int n, int lane, float* score, int stride, bool one_entry) {
    const bool valid = lane < n && doc >= 0 && doc < stride;
    const int d = valid ? doc : -1;
    if (one_entry) {
        if (valid) score[d] += m;
        return;
    }
    bool first = valid;
    float sum = m;
    for (int j = 0; j < n; ++j) {
        const int dj = __builtin_amdgcn_readlane(d, j);
        const float mj = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, m), j));
        if (dj == d) {
            if (j < lane) first = false;
            else if (j > lane) sum += mj;
        }
    }
    if (first) score[d] += sum;
}
constexpr int kMassStage = 4096;            // floats of partials staged per round by the stand-alone mass kernel

template <class T, class F>
__device__ __forceinline__ void segment_masses_block(const Plan& p, const SegTable& tbl, T* parts, T* stage,
                                                     MassScratch<T>* ms, F on_mass) {
    const int tid = threadIdx.x, nthr = blockDim.x;
    const unsigned total = (unsigned)tbl.tile0[tbl.n];
    const unsigned nsub = (unsigned)(p.nsplit * p.groups);
    const int nparts = p.units_per_b * p.nrb;
    constexpr int kGroup = 8;
    if (stage == nullptr) {                          // partials already in LDS: one thread per (group, column), in place
        const int ngroups = (nparts + kGroup - 1) / kGroup;
        for (int idx = tid; idx < ngroups * p.slots; idx += nthr) {
            const int g = (int)div_exact((unsigned)idx, (unsigned)p.slots), k = idx - g * p.slots;
            const T gs = group_sum(parts + g * kGroup * p.slots + k, p.slots, min(kGroup, nparts - g * kGroup));
            parts[g * kGroup * p.slots + k] = gs;
        }
        __syncthreads();
        for (int k = tid; k < p.slots; k += nthr) {
            T c = 0;
            for (int g = 0; g < ngroups; ++g) c += parts[g * kGroup * p.slots + k];
            ms->colsum[k] = c;
        }
    } else {                                         // partials in memory: whole rows through LDS, many loads in flight
        const int rows = kMassStage / p.slots / kGroup * kGroup;   // slots <= kMassStage / kGroup: whole groups per round
        T c[2] = {0, 0};                             // this thread's columns tid, tid + nthr (slots <= 2 * nthr)
        for (int r0 = 0; r0 < nparts; r0 += rows) {
            const int nr = min(rows, nparts - r0);
            __syncthreads();
            for (int i = tid; i < nr * p.slots; i += nthr) stage[i] = parts[(int64_t)r0 * p.slots + i];
            __syncthreads();
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int k = tid + j * nthr;
                if (k < p.slots)
                    for (int g0 = 0; g0 < nr; g0 += kGroup) c[j] += group_sum(stage + g0 * p.slots + k, p.slots, min(kGroup, nr - g0));
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (tid + j * nthr < p.slots) ms->colsum[tid + j * nthr] = c[j];
    }
    for (int sp = tid; sp <= (int)nsub; sp += nthr) ms->sub_begin[sp] = split_begin(total, nsub, sp);
    __syncthreads();
    for (int s = tid; s < tbl.n; s += nthr) {
        const int ts = tbl.tile0[s], te = tbl.tile0[s + 1];
        T m = 0;
        if (te > ts) {
            const int s0 = split_of(total, nsub, ts), s1 = split_of(total, nsub, te - 1);
            for (int sp = s0; sp <= s1; ++sp)
                if (ms->sub_begin[sp] < ms->sub_begin[sp + 1]) m += ms->colsum[s + sp];
        }
        on_mass(s, (float)m);
    }
}

// The runs of tiles that segment `lane` has tiles in: s0 .. s1 (none: s1 < s0), of those the ones in owns_mask (a split between a segment's first
// and last may own no tile at all).  span: the largest s1 - s0.
struct SegmentRuns { int s0, s1, span; unsigned long long owns_mask; };
__device__ __forceinline__ SegmentRuns segment_runs(const RegSegTable& t, unsigned nsub, int lane) {
    const unsigned total = (unsigned)t.total;
    SegmentRuns r;
    r.s0 = 0;
    r.s1 = -1;
    const bool has_tiles = lane < t.n && t.t1 > t.t0;
    bool owns;
    if (total < (1u << 14)) {                        // (nsub <= 64: every product below 2^21) the divisions side by side, their reciprocals shared
        const float per_total = __builtin_amdgcn_rcpf((float)total), per_nsub = __builtin_amdgcn_rcpf((float)nsub);
        const unsigned first = div_small(total * lane, nsub, per_nsub), next = div_small(total * (lane + 1), nsub, per_nsub);
        const unsigned s0 = div_small((t.t0 + 1) * nsub - 1, total, per_total), s1 = div_small(max(t.t1 * (int)nsub, 1) - 1, total, per_total);
        owns = lane < (int)nsub && first < next;
        if (has_tiles) { r.s0 = (int)s0; r.s1 = (int)s1; }
    } else {
        owns = lane < (int)nsub && split_begin(total, nsub, lane) < split_begin(total, nsub, lane + 1);
        if (has_tiles) { r.s0 = split_of(total, nsub, t.t0); r.s1 = split_of(total, nsub, t.t1 - 1); }
    }
    r.owns_mask = __ballot(owns);
    r.span = wave_max_i32(r.s1 - r.s0);
    return r;
}

// The same for one wavefront on its own, for a query with at most 128 slots and a register table: lane k adds
// up columns k and k + 64, lane s then collects segment s's slots — the same sums in the same order, no barrier.
// Returns lane s's segment mass (0 for lanes past the table).
// BATCHED: a column of at most 40 parts is requested in one batch (clamped, unconditional loads) before the first
// add, instead of a round trip — to memory or to LDS — per group of eight.
template <bool BATCHED = false, class T = float>
__device__ __forceinline__ float segment_masses_wave(const Plan& p, const RegSegTable& t, const T* parts, int lane) {
    const unsigned nsub = (unsigned)(p.nsplit * p.groups);
    const int nparts = p.units_per_b * p.nrb;
    constexpr int kGroup = 8;
    T c[2] = {0, 0};                                 // columns lane, lane + 64
    int first_looped = 0;
    if constexpr (BATCHED) {
        constexpr int kBatch = 40;
        if (nparts <= kBatch) {
            T v[kBatch];
            const T* col = parts + min(lane, p.slots - 1);
#pragma unroll
            for (int i = 0; i < kBatch; ++i) v[i] = col[min(i, nparts - 1) * p.slots];
            if (lane < p.slots) {
#pragma unroll
                for (int g0 = 0; g0 < kBatch; g0 += kGroup) {
                    T gs = 0;                        // the same sums in the same order as group_sum
#pragma unroll
                    for (int i = 0; i < kGroup; ++i)
                        if (g0 + i < nparts) gs += v[g0 + i];
                    if (g0 < nparts) c[0] += gs;
                }
            }
            first_looped = 1;
        }
    }
    for (int j = first_looped; j < 2; ++j)
        if (lane + 64 * j < p.slots)
            for (int g0 = 0; g0 < nparts; g0 += kGroup)
                c[j] += group_sum(parts + g0 * p.slots + lane + 64 * j, p.slots, min(kGroup, nparts - g0));
    const SegmentRuns r = segment_runs(t, nsub, lane);
    const unsigned long long owns_mask = r.owns_mask;
    const bool has_tiles = r.s1 >= r.s0;
    const int s0 = r.s0, s1 = r.s1, span = r.span;
    T m = 0;
    for (int d = 0; d <= span; ++d) {
        const int sp = s0 + d;
        const int slot = lane + sp;                                  // slot = segment + sub-split, < 128
        const T c_lo = __shfl(c[0], slot & (kWave - 1)), c_hi = __shfl(c[1], slot & (kWave - 1));
        if (has_tiles && sp <= s1 && ((owns_mask >> sp) & 1)) m += slot < kWave ? c_lo : c_hi;
    }
    return lane < t.n ? (float)m : 0.f;
}

// Third kernel: per-segment attention mass, one workgroup per query; then S += mass.
// Takes parts 0 .. n_parts - 1 of the ledger in order; the last one's masses go to `mass` when `write_mass` is set
// (it is not when only layers that deferred their scores are taken in, ahead of the fused epilogue).
// T: the type of the slot partials (double on the path that keeps fp32 precision throughout).
template <class T>
__global__ __launch_bounds__(kThreads) void attn_mass_kernel(AttnArgs a, Plan p, int n_parts, int write_mass) {
    __shared__ SegTable tbl;
    __shared__ MassScratch<T> ms;
    __shared__ T stage[kMassStage];
    const char* ws = static_cast<const char*>(a.workspace);
    const int b = __builtin_amdgcn_readfirstlane(blockIdx.x);
    const int tid = threadIdx.x;
    const int n_part_floats = p.units_per_b * p.nrb * p.slots;
    // part j of the ledger: the slot partials of the j-th layer still pending (the last one is this call's)
    auto part = [&](int j) { return reinterpret_cast<const T*>(ws + p.off_masspart + (size_t)j * p.masspart_bytes) + (int64_t)b * n_part_floats; };
    if (p.slots <= 2 * kWave && a.seg_stride <= kWave && n_part_floats <= kMassStage) {
        // small query: the partials go to LDS in one batch (requested before the query's scalars are waited for),
        // then one wavefront finishes alone from a table in its registers — the same sums in the same order
        T r_part[kMassStage / kThreads];
        const T* mp0 = part(0);
#pragma unroll
        for (int i = 0; i < kMassStage / kThreads; ++i) r_part[i] = mp0[min(tid + i * kThreads, n_part_floats - 1)];   // unconditional
        const QueryHead qh = load_query_head(a, b, tid & (kWave - 1));
#pragma unroll
        for (int i = 0; i < kMassStage / kThreads; ++i)
            if (tid + i * kThreads < n_part_floats) stage[tid + i * kThreads] = r_part[i];
        __syncthreads();
        if (n_parts == 1 && tid >= kWave) return;    // the other wavefronts only help to fetch further parts
        const RegSegTable rtbl = build_reg_table(a, qh, tid & (kWave - 1), p.tile);
        for (int j = 0; j < n_parts; ++j) {
            if (j > 0) {
                __syncthreads();                     // the staged part has been read
                const T* mp = part(j);
                for (int i = tid; i < n_part_floats; i += kThreads) stage[i] = mp[i];
                __syncthreads();
            }
            if (tid < kWave) {
                const float m = segment_masses_wave<false>(p, rtbl, stage, tid);
                if (write_mass && j == n_parts - 1 && tid < rtbl.n) a.mass[(int64_t)b * a.seg_stride + tid] = m;
                if (a.score_accum)                   // qh.seg is this lane's entry
                    add_doc_scores_wave(qh.seg.doc, m, rtbl.n, tid, a.score_accum + (int64_t)b * a.score_stride, a.score_stride,
                                        one_entry_per_slot(qh.seg.doc, rtbl.n, tid, a.score_stride));
            }
        }
        return;
    }
    const QueryHead qh = load_query_head(a, b, (int)threadIdx.x);
    build_table(a, qh, &tbl, p.tile);
    for (int j = 0; j < n_parts; ++j) {
        const bool last = write_mass && j == n_parts - 1;
        segment_masses_block(p, tbl, const_cast<T*>(part(j)), stage, &ms, [&](int s, float m) {
            if (last) a.mass[(int64_t)b * a.seg_stride + s] = m;
            ms.seg_mass[s] = m;
        });
        if (a.score_accum == nullptr) continue;
        __syncthreads();
        add_doc_scores_block(tbl.doc, ms.seg_mass, tbl.n, a.score_accum + (int64_t)b * a.score_stride, a.score_stride);
        __syncthreads();
    }
}

// The same for a small query with several parts to take in (layers that deferred their scores): one wavefront per
// part works out that layer's masses straight from the ledger, all parts at once; the first wavefront then adds them
// to the scores part by part — S += s^l in layer order, each document slot by the lane of its first table entry, so
// the sums are those of the one-part-after-the-other form above, bit for bit.  Any whole number of wavefronts per block;
// with fewer wavefronts than parts a wavefront takes several parts, one after the other.
__device__ __forceinline__ void pending_masses_block(const AttnArgs& a, const Plan& p, int b, int n_parts, int write_mass,
                                                     float (*m_all)[kWave]) {
    const char* ws = static_cast<const char*>(a.workspace);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int n_waves = (int)blockDim.x / kWave;
    const int n_part_floats = p.units_per_b * p.nrb * p.slots;
    const QueryHead qh = load_query_head(a, b, lane);
    const RegSegTable rtbl = build_reg_table(a, qh, lane, p.tile);
    for (int part = wave; part < n_parts; part += n_waves) {
        const float* mp = reinterpret_cast<const float*>(ws + p.off_masspart + (size_t)part * p.masspart_bytes) + (int64_t)b * n_part_floats;
        const float m = segment_masses_wave<true>(p, rtbl, mp, lane);
        m_all[part][lane] = m;
        if (write_mass && part == n_parts - 1 && lane < rtbl.n) a.mass[(int64_t)b * a.seg_stride + lane] = m;
    }
    __syncthreads();
    if (wave != 0 || a.score_accum == nullptr) return;
    // which entries feed this lane's document slot, and whether this lane is the slot's first entry: as in
    // add_doc_scores_wave, with the table walked once for all parts
    const int doc = qh.seg.doc;
    const bool valid = lane < rtbl.n && doc >= 0 && doc < a.score_stride;
    const int d = valid ? doc : -1;
    bool first = valid;
    unsigned long long later = 0;                    // entries after this one that feed the same slot
    for (int j = 0; j < rtbl.n; ++j) {
        const int dj = __builtin_amdgcn_readlane(d, j);
        if (dj == d) {
            if (j < lane) first = false;
            else if (j > lane) later |= 1ull << j;
        }
    }
    if (!first) return;
    float* slot = a.score_accum + (int64_t)b * a.score_stride + d;
    float s = *slot;
    for (int part = 0; part < n_parts; ++part) {
        float sum = m_all[part][lane];
        for (unsigned long long rest = later; rest; rest &= rest - 1) sum += m_all[part][__builtin_ctzll(rest)];
        s += sum;
    }
    *slot = s;
}

__global__ __launch_bounds__(kWave * (kMaxPending + 1)) void pending_masses_kernel(AttnArgs a, Plan p, int n_parts, int write_mass) {
    __shared__ float m_all[kMaxPending + 1][kWave];
    pending_masses_block(a, p, __builtin_amdgcn_readfirstlane(blockIdx.x), n_parts, write_mass, m_all);
}

// Fused layer epilogue (third kernel of cf_prefill_layer): one workgroup per query computes the
// attention mass of every segment (fixed summation order), adds it to the accumulated scores, and — when a prune step is attached —
// ranks the candidates, allocates the survivors' positions and writes the next layer's segment
// table, i.e. Alg. 2's "S += s; ids_sort = argsort(S); ids = prun(ids_sort)" followed by the
// allocation of Sec. 2.5, without leaving the GPU.
constexpr int kEpiThreads = 1024;
constexpr int kPartRegs = 8;                         // slot partials that a thread adds up


struct PruneArgs {
    int32_t enabled, keep, strategy, force_n_reuse, normalise_by_len, stride, pos_begin, pos_end, prefix_len,
        doc_stored_start;
    const int64_t* doc_tok_offset;
    const int32_t* doc_len;
    const int32_t* cand;
    const int32_t* n_cand;
    int32_t* keep_idx;
    int32_t* n_keep;
    int32_t* new_start;
    int32_t* q_start;
    int32_t* n_reuse;
    int32_t* order;
    cf_segment* next_segs;
    int32_t* next_n_seg;
};

// Every per-document row of the query (scores, lengths, candidates, offsets, positions) and the slot
// partial masses are fetched into LDS in one batch at the start: the ranking, the allocation and the
// table rebuild then run out of LDS with workgroup barriers between them instead of a round trip
// through memory per stage, and the results are written back at the end.
// Dynamic LDS: 44*stride + sizeof(T)*parts*slots bytes; larger problems take the stand-alone kernels.
// Bound by one wavefront's chain of instructions behind two round trips; what does not belong to the chain is the other wavefronts' (the slot
// partials' groups, each summed by the thread that read them, the look over the document slots, the ranking, the scores' way back).  One query, ten
// documents x 32 heads 13300 -> 10800 cycles, 50 documents x 4 heads 17700 -> 13100 (whole layers 20.5 -> 19.7 us and 34.0 -> 32.5).
// MORE: a small query with more group sums than threads, which the third wavefront and those after it take a second one of (a loop that the
// others' queries do not meet cost them 0.1 us).  32 heads, 300 query rows, 50 | 60 documents, 1440 | 1680 sums: with one wavefront adding them up
// 11.2 | 14.5 us, by the block functions 13.0 | 14.6, this way 6.3 | 6.4 (whole layers 57.9 | 58.4, 58.6 | 57.9 and 51.7 | 49.3).
template <class T, bool MORE>
__global__ __launch_bounds__(kEpiThreads) void layer_epilogue_kernel(AttnArgs a, Plan p, PruneArgs pr) {
    extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
    __shared__ SegTable tbl;
    __shared__ MassScratch<T> ms;
    __shared__ int s_int[7];
    __shared__ int32_t s_rank[kWave];

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int stride = pr.stride;
    int64_t* l_tok = reinterpret_cast<int64_t*>(dyn_smem);
    unsigned char* scratch = dyn_smem + (size_t)8 * stride;            // 3*stride words for ranking / allocation
    float* l_score = reinterpret_cast<float*>(scratch + (size_t)12 * stride);
    int32_t* l_len = reinterpret_cast<int32_t*>(l_score + stride);
    int32_t* l_cand = l_len + stride;
    int32_t* l_keep = l_cand + stride;
    int32_t* l_start = l_keep + stride;
    int32_t* l_order = l_start + stride;
    T* l_part = reinterpret_cast<T*>(dyn_smem + (((size_t)44 * stride + 7) & ~(size_t)7));

    const char* ws = static_cast<const char*>(a.workspace);
    const int b = __builtin_amdgcn_readfirstlane(blockIdx.x);
    const int64_t off = (int64_t)b * stride;
    const int nparts = p.units_per_b * p.nrb;
    // this call's own slot partials are part n_pending of the ledger (earlier parts, of layers that deferred their
    // scores, have been taken in by the mass kernel before this one)
    const T* mp_b = reinterpret_cast<const T*>(ws + p.off_masspart + (size_t)a.n_pending * p.masspart_bytes) + (int64_t)b * nparts * p.slots;
    // The first batch of row loads, the slot partials and the query's scalars all go out before anything is waited
    // for; every load is unconditional (a clamped, in-bounds index: threads past the end re-read the last element and
    // drop it), since a load inside a branch is waited for before the branch ends.
    const bool row0 = tid < stride;
    const int row_i = min(tid, stride - 1);
    const int64_t r_tok = pr.doc_tok_offset[off + row_i];
    const int32_t r_len = pr.doc_len[off + row_i], r_cand = pr.cand[off + row_i];
    const float r_score = a.score_accum[off + row_i];
    const int32_t r_start = pr.new_start[off + row_i], r_order = pr.order[off + row_i];
    // Slot partials, eight per thread.  Small queries: thread g * slots + k adds up group g of column k in its registers (the groups of
    // segment_masses_block).  Others: one after the other, to LDS.
    const int n_part_floats = nparts * p.slots;
    const int ngroups = (nparts + kPartRegs - 1) / kPartRegs;
    const int n_sums = ngroups * p.slots;
    const bool grouped = p.slots <= 2 * kWave && a.seg_stride <= kWave;
    const int part_g = grouped ? (int)div_exact((unsigned)tid, (unsigned)p.slots) : 0, part_k = tid - part_g * p.slots;
    const int part_first = grouped ? part_g * kPartRegs * p.slots + part_k : tid, part_step = grouped ? p.slots : kEpiThreads;
    const int part_last = grouped ? (nparts - 1) * p.slots + part_k : n_part_floats - 1;
    T r_part[kPartRegs];
#pragma unroll
    for (int i = 0; i < kPartRegs; ++i) r_part[i] = mp_b[min(part_first + i * part_step, part_last)];
    const int n_cand = pr.n_cand[b];
    const int r_q_start = pr.q_start[b], r_n_reuse = pr.n_reuse[b];
    const QueryHead qh = load_query_head(a, b, grouped ? lane : tid);
    if (tid == 0) { s_int[4] = r_q_start; s_int[5] = r_n_reuse; }
    if (tid < kWave) s_rank[tid] = 0;
    if (row0) {
        l_tok[tid] = r_tok; l_len[tid] = r_len; l_cand[tid] = r_cand; l_score[tid] = r_score; l_start[tid] = r_start;
        l_order[tid] = r_order;
    }
    for (int i = tid + kEpiThreads; i < stride; i += kEpiThreads) {
        l_tok[i] = pr.doc_tok_offset[off + i];
        l_len[i] = pr.doc_len[off + i];
        l_cand[i] = pr.cand[off + i];
        l_score[i] = a.score_accum[off + i];
        l_start[i] = pr.new_start[off + i];
        l_order[i] = pr.order[off + i];
    }
    // With few candidates one wavefront finishes alone: the others leave, and the barriers of the stages
    // below (which only wait for wavefronts that are still running) cost nothing.
    const int nthr = n_cand <= 2 * kWave ? kWave : kEpiThreads;
    const bool small = nthr == kWave && grouped;
    SelectWaveArgs sw;
    sw.score = l_score; sw.len = l_len; sw.cand = l_cand; sw.tok = l_tok; sw.start = l_start;
    sw.keep_idx = pr.keep_idx + off; sw.new_start = pr.new_start + off; sw.order = pr.order + off;
    sw.n = n_cand; sw.keep = pr.keep; sw.stride = stride; sw.normalise_by_len = pr.normalise_by_len;
    sw.strategy = pr.strategy; sw.force_n_reuse = pr.force_n_reuse; sw.pos_begin = pr.pos_begin; sw.pos_end = pr.pos_end;
    sw.prefix_len = pr.prefix_len; sw.doc_stored_start = pr.doc_stored_start; sw.q_stored_start = a.q_stored_start;
    sw.q_lo = qh.q0; sw.q_hi = qh.q0 + qh.tq_raw; sw.seg_stride = a.seg_stride; sw.q_start = r_q_start; sw.n_reuse = r_n_reuse;
    RankShare share;
    if (small) {
        // Small query: the first wavefront does the masses, from a table in its registers, the second one looks the document slots over.
        T gs = 0;
#pragma unroll
        for (int i = 0; i < kPartRegs; ++i)
            if (part_g * kPartRegs + i < nparts) gs += r_part[i];
        if (tid < n_sums) l_part[tid] = gs;
        if constexpr (MORE) {
            for (int x = kEpiThreads + tid - 2 * kWave; wave >= 2 && x < n_sums; x += kEpiThreads - 2 * kWave) {
                const int g = (int)div_exact((unsigned)x, (unsigned)p.slots), first = g * kPartRegs, k = x - g * p.slots;
                T v[kPartRegs], sum = 0;
#pragma unroll
                for (int i = 0; i < kPartRegs; ++i) v[i] = mp_b[min(first + i, nparts - 1) * p.slots + k];
#pragma unroll
                for (int i = 0; i < kPartRegs; ++i)
                    if (first + i < nparts) sum += v[i];
                l_part[x] = sum;
            }
        }
        RegSegTable rtbl;
        SegmentRuns runs;
        unsigned long long mine = 0;                 // bit i: run s0 + i is the segment's
        if (wave == 0) {
            rtbl = build_reg_table(a, qh, lane, p.tile);
            runs = segment_runs(rtbl, (unsigned)(p.nsplit * p.groups), lane);
            if (runs.s1 >= runs.s0) mine = (runs.owns_mask >> runs.s0) & (~0ull >> (63 - (runs.s1 - runs.s0)));
        } else if (wave == 1) {
            const bool one = one_entry_per_slot(qh.seg.doc, qh.n_seg < 0 ? 0 : min(qh.n_seg, a.seg_stride), lane, stride);
            if (lane == 0) s_int[6] = one;
        }
        __syncthreads();                             // publishes the rows and the groups' sums
        if (wave > 0 && n_cand <= kWave) share = rank_prepare(sw, wave - 1, kEpiThreads / kWave - 1);
        if (wave == 0) {
            // the sums of segment_masses_wave in the same order; columns to LDS, a segment's come from there
            T c[2] = {0, 0};
            for (int g0 = 0; g0 < ngroups; g0 += 4) {
                T v[2][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int at = min(g0 + i, ngroups - 1) * p.slots;
                    v[0][i] = l_part[at + min(lane, p.slots - 1)];
                    v[1][i] = l_part[at + min(lane + kWave, p.slots - 1)];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (g0 + i < ngroups) { c[0] += v[0][i]; c[1] += v[1][i]; }
            }
            ms.colsum[lane] = c[0];
            ms.colsum[lane + kWave] = c[1];
            wave_lds_order();
            T m = 0;
            for (int d0 = 0; d0 <= runs.span; d0 += 4) {
                T v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = ms.colsum[min(lane + runs.s0 + d0 + i, 2 * kWave - 1)];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if ((uint32_t)mine >> i & 1) m += v[i];
                mine >>= 4;
            }
            if (lane < rtbl.n) a.mass[(int64_t)b * a.seg_stride + lane] = (float)m;
            add_doc_scores_wave(qh.seg.doc, lane < rtbl.n ? (float)m : 0.f, rtbl.n, lane, l_score, stride, s_int[6] != 0);      // qh.seg is this lane's entry
        }
        __syncthreads();
    } else {
        if (grouped) {
            for (int i = tid; i < n_part_floats; i += kEpiThreads) l_part[i] = mp_b[i];
        } else {
#pragma unroll
            for (int i = 0; i < kPartRegs; ++i)
                if (tid + i * kEpiThreads < n_part_floats) l_part[tid + i * kEpiThreads] = r_part[i];
            for (int i = tid + kPartRegs * kEpiThreads; i < n_part_floats; i += kEpiThreads) l_part[i] = mp_b[i];
        }
        build_table(a, qh, &tbl, p.tile);            // its barriers also publish the rows above
        segment_masses_block<T>(p, tbl, l_part, nullptr, &ms, [&](int s, float m) {
            a.mass[(int64_t)b * a.seg_stride + s] = m;
            ms.seg_mass[s] = m;
        });
        __syncthreads();
        add_doc_scores_block(tbl.doc, ms.seg_mass, tbl.n, l_score, stride);
        __syncthreads();
    }
    Candidate cand;
    if (n_cand <= kWave) {                               // the usual case: everything in registers
        if (wave > 0) {
            if (!small) share = rank_prepare(sw, wave - 1, kEpiThreads / kWave - 1);
            rank_share(sw, share, s_rank);
        } else {
            cand = load_candidate(sw);
        }
        __syncthreads();
    }
    // (by the others, where the first wavefront goes on alone)
    const int first_writer = nthr == kWave ? kWave : 0;
    if (tid >= first_writer)
        for (int i = tid - first_writer; i < stride; i += kEpiThreads - first_writer) a.score_accum[off + i] = l_score[i];
    if (tid >= nthr) return;
    if (n_cand <= kWave &&
        select_wave64(sw, cand, s_rank[lane], pr.n_keep + b, pr.q_start + b, pr.n_reuse + b, pr.next_segs + (int64_t)b * a.seg_stride, pr.next_n_seg + b))
        return;
    const int k = prune_topk_block(l_score, pr.normalise_by_len ? l_len : nullptr, l_cand, n_cand, pr.keep, stride, l_keep, a.dev_flag, scratch, &s_int[3],
                                   nthr);
    if (tid == 0) pr.n_keep[b] = k;
    __syncthreads();
    assign_positions_block(l_len, l_keep, k, stride, pr.pos_begin, pr.pos_end, pr.strategy, pr.force_n_reuse, l_start, &s_int[4], &s_int[5], l_order,
                           a.dev_flag, scratch, s_int, nthr);
    __syncthreads();
    gather_segments_block(l_tok, l_len, l_order, k, l_start, s_int[4], qh.q0, qh.q0 + qh.tq_raw, stride, pr.prefix_len, pr.doc_stored_start,
                          a.q_stored_start, pr.next_segs + (int64_t)b * a.seg_stride, pr.next_n_seg + b, a.seg_stride, a.dev_flag, nthr);
    for (int i = tid; i < stride; i += nthr) {
        if (i < k) pr.keep_idx[off + i] = l_keep[i];
        pr.new_start[off + i] = l_start[i];
        pr.order[off + i] = l_order[i];
    }
    if (tid == 0) { pr.q_start[b] = s_int[4]; pr.n_reuse[b] = s_int[5]; }
}

}  // namespace

bool pending_fit_combine(const AttnArgs& a, const Plan& p) { return p.slots <= 2 * kWave && a.seg_stride <= kWave; }

template <int DT, int NS>
static void launch_combine_ns(const AttnArgs& a, const Plan& p, int extra, hipStream_t s) {
    const int spread = p.nrb > 1 || p.blocks_rg > 2 ? 0 : p.blocks_rg == 2 ? 1 : 2;
    const dim3 grid((unsigned)p.units_per_b, (unsigned)((8 >> spread) * p.nrb + extra), (unsigned)a.batch), block(kThreads);
    if (a.mass != nullptr) hipLaunchKernelGGL((attn_combine_kernel<DT, NS, true>), grid, block, 0, s, a, p, extra, spread);
    else hipLaunchKernelGGL((attn_combine_kernel<DT, NS, false>), grid, block, 0, s, a, p, extra, spread);
}

void launch_combine(const AttnArgs& a, const Plan& p, bool take_pending, hipStream_t s) {
    const int extra = take_pending ? 1 : 0;
    auto by_splits = [&](auto dt) {
        constexpr int DT = decltype(dt)::value;
        if (p.nsplit <= 8) launch_combine_ns<DT, 8>(a, p, extra, s);
        else if (p.nsplit <= 16) launch_combine_ns<DT, 16>(a, p, extra, s);
        else launch_combine_ns<DT, kMaxSplit>(a, p, extra, s);
    };
    if (a.dtype == CF_BF16) by_splits(std::integral_constant<int, CF_BF16>{});
    else by_splits(std::integral_constant<int, CF_F16>{});
}

// several parts of a small query: one wavefront per part (see pending_masses_kernel); else one part after the other
static void launch_masses(const AttnArgs& a, const Plan& p, int n_parts, int write_mass, hipStream_t s) {
    if (n_parts > 1 && pending_fit_combine(a, p))
        hipLaunchKernelGGL(pending_masses_kernel, dim3((unsigned)a.batch), dim3(kWave * n_parts), 0, s, a, p, n_parts, write_mass);
    else
        hipLaunchKernelGGL(attn_mass_kernel<float>, dim3((unsigned)a.batch), dim3(kThreads), 0, s, a, p, n_parts, write_mass);
}

void launch_mass(const AttnArgs& a, const Plan& p, hipStream_t s) { launch_masses(a, p, a.n_pending + 1, 1, s); }

void launch_pending_masses(const AttnArgs& a, const Plan& p, hipStream_t s) { launch_masses(a, p, a.n_pending, 0, s); }

void launch_mass_f64(const AttnArgs& a, const Plan& p, hipStream_t s) {
    hipLaunchKernelGGL(attn_mass_kernel<double>, dim3((unsigned)a.batch), dim3(kThreads), 0, s, a, p, 1, 1);
}

static size_t epilogue_lds_bytes(const Plan& p, const cf_prune_step* prune, size_t elem) {
    return (((size_t)44 * prune->stride + 7) & ~(size_t)7) + elem * p.units_per_b * p.nrb * p.slots;
}

bool epilogue_fits(const Plan& p, const cf_prune_step* prune) { return epilogue_lds_bytes(p, prune, sizeof(float)) <= 60 * 1024; }
bool epilogue_fits_f64(const Plan& p, const cf_prune_step* prune) { return epilogue_lds_bytes(p, prune, sizeof(double)) <= 60 * 1024; }

static PruneArgs prune_args(const cf_prune_step* prune) {
    PruneArgs pr;
    pr.enabled = 1; pr.keep = prune->keep; pr.strategy = prune->strategy; pr.force_n_reuse = prune->force_n_reuse;
    pr.normalise_by_len = prune->normalise_by_len; pr.stride = prune->stride; pr.pos_begin = prune->pos_begin;
    pr.pos_end = prune->pos_end; pr.prefix_len = prune->prefix_len; pr.doc_stored_start = prune->doc_stored_start;
    pr.doc_tok_offset = prune->doc_tok_offset; pr.doc_len = prune->doc_len; pr.cand = prune->cand;
    pr.n_cand = prune->n_cand; pr.keep_idx = prune->keep_idx; pr.n_keep = prune->n_keep;
    pr.new_start = prune->new_start; pr.q_start = prune->q_start; pr.n_reuse = prune->n_reuse;
    pr.order = prune->order; pr.next_segs = prune->next_segs; pr.next_n_seg = prune->next_n_seg;
    return pr;
}

template <class T>
static void launch_epilogue_of(const AttnArgs& a, const Plan& p, const cf_prune_step* prune, hipStream_t s) {
    const int sums = (p.units_per_b * p.nrb + kPartRegs - 1) / kPartRegs * p.slots;
    const size_t lds = epilogue_lds_bytes(p, prune, sizeof(T));
    if (sums > kEpiThreads) hipLaunchKernelGGL((layer_epilogue_kernel<T, true>), dim3(a.batch), dim3(kEpiThreads), lds, s, a, p, prune_args(prune));
    else hipLaunchKernelGGL((layer_epilogue_kernel<T, false>), dim3(a.batch), dim3(kEpiThreads), lds, s, a, p, prune_args(prune));
}
void launch_epilogue(const AttnArgs& a, const Plan& p, const cf_prune_step* prune, hipStream_t s) { launch_epilogue_of<float>(a, p, prune, s); }
void launch_epilogue_f64(const AttnArgs& a, const Plan& p, const cf_prune_step* prune, hipStream_t s) { launch_epilogue_of<double>(a, p, prune, s); }

}  // namespace cf
