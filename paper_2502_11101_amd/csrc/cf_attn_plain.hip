// Prefill attention for everything the 16-bit kernels of cf_attn_mfma.hip do not serve: fp32 tensors, head sizes other
// than 128, interleaved RoPE pairs.  Every step keeps fp32 precision, whatever the tensors' type.
//
// Work decomposition, as in cf_attn_mfma.hip: the query rows that share a kv head are stacked and cut into 16-row
// blocks; a workgroup of four wavefronts owns RB of them (1, 2 or 4) and a run of the attended tokens.  The wavefronts form 4 / RB
// groups; a group streams tiles of its own (16 tokens of fp32, 32 of a 16-bit type), a wavefront of it owns one row block, and the groups
// merge through LDS at the end — so a short query fills the workgroup with tokens where it has no rows.
//
// Precision and where the rotation happens.  q . (R_d k) = (R_-d q) . k (Eq. 2), so the query rows are turned by the segment's
// relative shift once per segment, in fp32, and keys and values go to LDS as they are: no arithmetic per cached token.
//   * fp32: S^T = K Q^T and O^T += V^T P^T on v_mfma_f32_16x16x4f32.
//   * bf16 / fp16: keys and values are exact MFMA operands; the turned query and the probabilities are fp32 numbers handed
//     over as sums of three 16-bit parts (bf16: 8 + 8 + 8 significant bits; fp16: 11 + 11 + 11, each part scaled up by 2^11
//     against the one before it so that none underflows, with an accumulator per part).  Products of parts are exact
//     in the fp32 accumulators, so the result has fp32 precision at a third of the 16-bit matrix rate: 2048 -> 384 matrix cycles
//     per 16 rows x 32 tokens x 128 channels and product, against v_mfma_f32_16x16x4f32.
//
// Infinities and NaN: a tile's product multiplies the tokens a row does not see by zero, and parts do not add up to an infinity;
// rows whose sums are not finite at the end are gone over once more token by token (redo_row).
//
// Bound by the latency of a launch's memory round trips at the sizes measured: bf16, interleaved pairs, 32 heads, 10 documents of 100-200
// tokens, 48 query rows, eight splits: 17.4 us for 26.7 MB of keys, values, queries and outputs, the wavefronts waiting 51 % of their cycles,
// matrix pipe busy 11 %, VALU issue 21 %; the merge 4.4 us.  Whole layer calls with a prune event, from the row-by-row kernel of
// cf_attn_generic.hip to this one: 916 -> 26.8 us; fp32, head_dim 64, 4 heads, 4 x 32 tokens, 8 rows: 54 -> 16.2 us.  fp16 at the first one's
// shape takes 8 % more than bf16.
#include "cf_attn_plan.h"
#include "cf_attn_tile.h"

namespace cf {
using namespace attn;
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// workgroups that fit a CU, by registers and LDS
constexpr int plain_per_cu(bool f32, int dp, int rb) { return dp == 256 || (!f32 && dp == 128 && rb < 4) ? 1 : 2; }

// 16-byte chunks hold 4 fp32 or 8 16-bit channels.  A lane group lg takes, in step (g, h) of a score product, chunk
// 4*g + lg of the first (h = 0) or second half (h = 1) of the head: both members of a half-split pair sit in one lane.
template <int DT, int DP> struct PlainShape {
    static constexpr bool kF32 = DT == CF_F32;
    static constexpr int kEsz = kF32 ? 4 : 2;
    static constexpr int kTile = kF32 ? 16 : 32;
    static constexpr int kPerChunk = 16 / kEsz;
    static constexpr int kChunks = DP * kEsz / 16;           // per token row
    static constexpr int kSteps = kChunks / 8;               // pair groups g: four pairs of chunks each
    static constexpr int kKRow = DP * kEsz + 16;             // LDS bytes per key row: 16 rows' chunks fall into different banks
    static constexpr int kVRow = DP * kEsz + (kF32 ? 16 : 32);   // per value row: the rows of one (transposing) read likewise
    static constexpr int kBlocks = DP / 16;                  // 16-channel blocks of the output
    static constexpr int kBuf = kTile * (kKRow + kVRow);
    static constexpr int kQParts = kF32 ? 1 : 3;
    static constexpr int kPParts = 3;                        // 16-bit parts of a probability
};

// fp16 probabilities live in (0, 2^15]: the reference stays 2^7 below the row maximum it was taken from.  Three parts, the second
// and third scaled up by 2^11 and 2^22, hold all 24 bits of a probability down to 2^-30 of the largest, and 2^-53 of that at worst
template <int DT> constexpr float kRefBelow = DT == CF_F16 ? 7.f : 0.f;
template <int DT> constexpr float kPlainLimit = DT == CF_F16 ? 32768.f : kProbLimit;

template <int DT>
__device__ __forceinline__ void unpack_chunk(uint4 w, float (&v)[8]) {
    const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (DT == CF_F32) v[i] = __uint_as_float(u[i]);
        else { v[2 * i] = Mma<DT>::lo(u[i]); v[2 * i + 1] = Mma<DT>::hi(u[i]); }
    }
}

// the leading 16-bit part of eight fp32 values, which keep the rest (times `up`)
template <int DT>
__device__ __forceinline__ uint4 split_part(float (&v)[8], float up) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w[i] = Mma<DT>::pack(v[2 * i], v[2 * i + 1]);
        v[2 * i] = (v[2 * i] - Mma<DT>::lo(w[i])) * up;
        v[2 * i + 1] = (v[2 * i + 1] - Mma<DT>::hi(w[i])) * up;
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// Turns a lane's chunks by (cos, sin) pairs of a segment: half-split pairs lie in the chunks x and y of one step, interleaved
// ones inside each chunk.  cs_x, cs_y: the pairs of x's slices (half-split) or of x's and y's (interleaved).
template <int N>
__device__ __forceinline__ void turn_chunks(float (&x)[8], float (&y)[8], const float2* cs_x, const float2* cs_y, bool interleaved) {
    if (!interleaved) {
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const float2 w = cs_x[e];
            const float nx = x[e] * w.x + y[e] * w.y;
            y[e] = y[e] * w.x - x[e] * w.y;
            x[e] = nx;
        }
    } else {
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
            const float2 u = cs_x[i], w = cs_y[i];
            const float x0 = x[2 * i] * u.x + x[2 * i + 1] * u.y, y0 = y[2 * i] * w.x + y[2 * i + 1] * w.y;
            x[2 * i + 1] = x[2 * i + 1] * u.x - x[2 * i] * u.y;
            y[2 * i + 1] = y[2 * i + 1] * w.x - y[2 * i] * w.y;
            x[2 * i] = x0;
            y[2 * i] = y0;
        }
    }
}

// A row's weight on a slot: (reference, sum) of the slot against those of the row, divided in double.
__device__ __forceinline__ double slot_share(float2 v, float2 row) {
    return row.y > 0.f && v.y > 0.f ? (double)(v.y * exp2f(v.x - row.x)) / (double)row.y : 0.0;
}

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

template <int DT, int DP, int RB>
__global__ __launch_bounds__(kThreads, plain_per_cu(DT == CF_F32, DP, RB)) void attn_plain_kernel(AttnArgs a, RopeFreq freq, Plan p) {
    using S = PlainShape<DT, DP>;
    constexpr int kGroups = kWaves / RB;
    constexpr int kGroupThreads = kWave * RB;
    constexpr int kBufs = 2 * kGroups * S::kBuf <= 72 * 1024 ? 2 : 1;       // two tile buffers where two workgroups still fit a CU
    constexpr int kItems = S::kTile * S::kChunks / kGroupThreads;           // 16-byte chunks per thread and tensor
    __shared__ SegTable tbl;
    __shared__ __attribute__((aligned(16))) unsigned char bufs[kGroups][kBufs][S::kBuf];
    __shared__ __attribute__((aligned(16))) float2 cs_lds[kGroups][3][DP / 2];
    __shared__ float2 ml_lds[kGroups][16 * RB];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave_all = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int grp = wave_all / RB, wave = wave_all % RB;     // group, row block of this wavefront
    const int tid = threadIdx.x & (kGroupThreads - 1);       // thread of the group
    const int li = lane & 15, lg = lane >> 4;

    // grid (split, kv head * row groups + row group, query)
    const int split = blockIdx.x, b = blockIdx.z;
    const int hkv = p.n_rg == 1 ? (int)blockIdx.y : (int)div_exact(blockIdx.y, (unsigned)p.n_rg);
    const int rg = (int)blockIdx.y - hkv * p.n_rg;
    const int unit = b * p.units_per_b + (int)blockIdx.y;
    const int d = a.head_dim, group = p.group;
    const int n_pairs = d / (2 * S::kPerChunk);              // chunk pairs of a row: chunks j and j + n_pairs
    const bool reg_table = a.seg_stride <= kWave;
    const QueryHead qh = load_query_head(a, b, reg_table ? lane : (int)threadIdx.x);
    // requested with the table: read where a segment begins, each segment waited a round trip more for it (4 x 32 tokens x 4 heads in
    // fp32 12.8 -> 12.2 us, 10 documents x 32 heads 18.1 -> 17.1)
    static_assert(DP / 2 <= kGroupThreads, "a thread has at most one slice");
    const double my_freq = freq.rev[min(tid, DP / 2 - 1)];
    const int tq = min(qh.tq_raw, a.max_tq);
    const int row_base = rg * p.blocks_rg * 16;
    const int row_limit = min(group * tq, row_base + p.blocks_rg * 16);
    const bool has_rows = row_base + wave * 16 < row_limit;  // wavefront-uniform
    const int m_row = row_base + wave * 16 + li;
    const bool row_ok = m_row < row_limit;
    const int gi = row_ok ? (int)div_exact((unsigned)m_row, (unsigned)tq) : 0;
    const int t_row = row_ok ? m_row - gi * tq : 0;
    const int trow = row_ok ? t_row : 0x7fffffff;            // padding rows mask nothing

    // the lane's raw query chunks (padding rows and chunks past the head: zero)
    uint4 qraw[S::kSteps][2];
    {
        const char* qp = static_cast<const char*>(a.q) + (((int64_t)qh.q0 + t_row) * a.n_q_heads + hkv * group + gi) * d * S::kEsz;
#pragma unroll
        for (int g = 0; g < S::kSteps; ++g)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = 4 * g + lg;
                qraw[g][h] = row_ok && j < n_pairs ? *reinterpret_cast<const uint4*>(qp + 16 * (j + h * n_pairs)) : make_uint4(0, 0, 0, 0);
            }
    }

    RegSegTable rtbl;
    unsigned total;
    if (reg_table) {
        rtbl = build_reg_table(a, qh, lane, S::kTile);
        total = (unsigned)rtbl.total;
    } else {
        rtbl = RegSegTable{};
        build_table(a, qh, &tbl, S::kTile);
        total = (unsigned)tbl.tile0[tbl.n];
    }
    const unsigned nsub = (unsigned)(p.nsplit * kGroups);
    const int ss = split * kGroups + grp;                    // the group's sub-split
    TileWalk<S::kTile> walk(split_begin(total, nsub, ss), split_begin(total, nsub, ss + 1));
    int most_tiles = 0;
#pragma unroll
    for (int g = 0; g < kGroups; ++g)
        most_tiles = max(most_tiles, split_begin(total, nsub, split * kGroups + g + 1) - split_begin(total, nsub, split * kGroups + g));

    // staging item i of a thread: row sr + i * rows per sweep, chunk sc (chunks past the head re-read its last one; nobody uses them)
    constexpr int kSweep = kGroupThreads / S::kChunks > 0 ? kGroupThreads / S::kChunks : 1;
    static_assert(kGroupThreads % S::kChunks == 0, "a sweep covers whole rows");
    const int sr = tid / S::kChunks, sc = tid % S::kChunks;
    const uint32_t sc_off = 16u * (uint32_t)min(sc, 2 * n_pairs - 1);
    // (a vector type of the language: structs that are only copied from memory to LDS would live in scratch memory)
    struct StageRegs { u32x4 k[kItems], v[kItems]; } regs;
    auto fetch = [&](Tile& t, StageRegs& r) __attribute__((always_inline)) {
        if (reg_table) t = walk.next(rtbl, lane);
        else t = walk.next(tbl, lane);
        const char *kp = static_cast<const char*>(a.workspace), *vp = kp;    // without a tile: something readable
        uint32_t row_bytes = 0, chunk = 0;
        int last = 0;
        if (t.ntok > 0) {
            const int64_t ts = t.self ? (int64_t)a.n_kv_heads * d : a.store_ts;      // the own block is always token-major
            const int64_t base = ((walk.c_tok + t.tok0) * ts + (int64_t)hkv * (t.self ? d : a.store_hs)) * S::kEsz;
            kp = static_cast<const char*>(t.self ? a.k_self : a.k_store) + base;
            vp = static_cast<const char*>(t.self ? a.v_self : a.v_store) + base;
            row_bytes = (uint32_t)ts * S::kEsz;
            last = t.ntok - 1;
            chunk = sc_off;
        }
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            const uint32_t off = (uint32_t)min(sr + i * kSweep, last) * row_bytes + chunk;
            r.k[i] = *reinterpret_cast<const u32x4*>(kp + off);
            r.v[i] = *reinterpret_cast<const u32x4*>(vp + off);
        }
    };
    auto make_angles = [&](const Tile& t, int slot) __attribute__((always_inline)) {
        if (tid < d / 2) cs_lds[grp][slot][tid] = rope_cos_sin(t.delta, my_freq);
    };

    // running state: O^T (channel 16*db + 4*lg + r of row li), softmax reference, sums over the lane's own tokens
    f32x4 acc[S::kBlocks];
#pragma unroll
    for (int db = 0; db < S::kBlocks; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f, seg_l = 0.f;
    // the turned query: fp32, or its 16-bit parts
    uint4 qt[S::kQParts][S::kSteps][2];
    bool turned = false;                                     // whether the current segment's query has parts past the first

    auto turn_query = [&](const Tile& t, int slot) __attribute__((always_inline)) {
        turned = t.delta != 0;
#pragma unroll
        for (int g = 0; g < S::kSteps; ++g) {
            if (!turned && DT != CF_F16) {                   // the query as it is
                qt[0][g][0] = qraw[g][0];
                qt[0][g][1] = qraw[g][1];
                continue;
            }
            float x[8], y[8];
            unpack_chunk<DT>(qraw[g][0], x);
            unpack_chunk<DT>(qraw[g][1], y);
            if (turned) {
                const float2* cs = cs_lds[grp][slot];
                const int j = min(4 * g + lg, n_pairs - 1);  // chunks past the head are zero and stay so
                const bool il = a.pairing != CF_ROPE_HALF;
                turn_chunks<S::kPerChunk>(x, y, cs + (il ? j * (S::kPerChunk / 2) : j * S::kPerChunk),
                                          cs + (il ? (j + n_pairs) * (S::kPerChunk / 2) : 0), il);
            }
            if constexpr (S::kF32) {
                qt[0][g][0] = make_uint4(__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3]));
                qt[0][g][1] = make_uint4(__float_as_uint(y[0]), __float_as_uint(y[1]), __float_as_uint(y[2]), __float_as_uint(y[3]));
            } else {
                constexpr float up = DT == CF_F16 ? 2048.f : 1.f;
                if constexpr (DT == CF_F16) {                // halved: a turned component may pass the type's range by sqrt(2)
#pragma unroll
                    for (int e = 0; e < 8; ++e) { x[e] *= 0.5f; y[e] *= 0.5f; }
                }
#pragma unroll
                for (int n = 0; n < S::kQParts; ++n) {
                    qt[n][g][0] = split_part<DT>(x, up);
                    qt[n][g][1] = split_part<DT>(y, up);
                }
            }
        }
        // (fp16: halving may drop the last bit of a subnormal, which the second part then holds)
        if constexpr (DT == CF_F16) turned = true;
    };
    const float scale = DT == CF_F16 ? 2.f * a.scale_log2e : a.scale_log2e;

    constexpr int kTok = S::kF32 ? 4 : 8;                    // tokens of a tile a lane holds: 16*tb + 4*lg + r
    auto tile_pass = [&](const Tile& cd, const unsigned char* k_lds, const unsigned char* v_lds) __attribute__((always_inline)) {
        float xv[kTok], pv[kTok];
        // ---- S^T = K Q^T
        if constexpr (S::kF32) {
            f32x4 s0 = f32x4{0.f, 0.f, 0.f, 0.f}, s1 = s0;   // two chains
#pragma unroll
            for (int g = 0; g < S::kSteps; ++g) {
                const int j = min(4 * g + lg, n_pairs - 1);
                const f32x4 ka = *reinterpret_cast<const f32x4*>(k_lds + li * S::kKRow + 16 * j);
                const f32x4 kb = *reinterpret_cast<const f32x4*>(k_lds + li * S::kKRow + 16 * (j + n_pairs));
                const f32x4 qa = __builtin_bit_cast(f32x4, qt[0][g][0]), qb = __builtin_bit_cast(f32x4, qt[0][g][1]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(ka[e], qa[e], s0, 0, 0, 0);
                    s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kb[e], qb[e], s1, 0, 0, 0);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) xv[e] = s0[e] + s1[e];
        } else {
            constexpr int kAccs = DT == CF_F16 ? 3 : 1;      // fp16: an accumulator per (scaled) part
            f32x4 s[kAccs][2];
#pragma unroll
            for (int n = 0; n < kAccs; ++n) { s[n][0] = f32x4{0.f, 0.f, 0.f, 0.f}; s[n][1] = s[n][0]; }
            auto steps = [&](auto parts_tag) __attribute__((always_inline)) {
                constexpr int kParts = decltype(parts_tag)::value;
#pragma unroll
                for (int g = 0; g < S::kSteps; ++g) {
                    const int j = min(4 * g + lg, n_pairs - 1);
                    uint4 kf[2][2];
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int tb = 0; tb < 2; ++tb)
                            kf[h][tb] = *reinterpret_cast<const uint4*>(k_lds + (16 * tb + li) * S::kKRow + 16 * (j + h * n_pairs));
#pragma unroll
                    for (int n = kParts - 1; n >= 0; --n)    // the small parts first
#pragma unroll
                        for (int h = 0; h < 2; ++h)
#pragma unroll
                            for (int tb = 0; tb < 2; ++tb)
                                s[kAccs == 1 ? 0 : n][tb] = Mma<DT == CF_F32 ? CF_BF16 : DT>::run(kf[h][tb], qt[n][g][h], s[kAccs == 1 ? 0 : n][tb]);
                }
            };
            if (turned) steps(std::integral_constant<int, S::kQParts>{});
            else steps(std::integral_constant<int, 1>{});
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float x = s[0][tb][e];
                    if constexpr (DT == CF_F16) x += (s[1][tb][e] + s[kAccs - 1][tb][e] * 0x1p-11f) * 0x1p-11f;
                    xv[4 * tb + e] = x;
                }
        }
        if (cd.ntok < S::kTile || cd.self) {
#pragma unroll
            for (int e = 0; e < kTok; ++e) {
                const int tk = 16 * (e >> 2) + 4 * lg + (e & 3);
                if (!(tk < cd.ntok && (!cd.self || cd.tok0 + tk <= trow))) xv[e] = -INFINITY;
            }
        }
        // ---- online softmax against a stale reference (see kProbLimit)
        float lsum;
        auto probabilities = [&](float m_ref) __attribute__((always_inline)) {
            const float m_safe = m_ref == -INFINITY ? 0.f : m_ref;
            lsum = 0.f;
#pragma unroll
            for (int e = 0; e < kTok; ++e) {
                pv[e] = __builtin_amdgcn_exp2f(fmaf(xv[e], scale, -m_safe));
                lsum += pv[e];
            }
        };
        probabilities(m_run);
        if (__any(!(lsum <= kPlainLimit<DT>) || m_run == -INFINITY)) {
            float mloc = xv[0];
#pragma unroll
            for (int e = 1; e < kTok; ++e) mloc = fmaxf(mloc, xv[e]);
            mloc = mloc * scale - kRefBelow<DT>;             // scale > 0: max commutes with it
            mloc = fmaxf(mloc, __shfl_xor(mloc, 16));
            mloc = fmaxf(mloc, __shfl_xor(mloc, 32));
            const float m_new = fmaxf(m_run, mloc);
            const float alpha = __builtin_amdgcn_exp2f(m_run - (m_new == -INFINITY ? 0.f : m_new));
            l_run *= alpha;
            seg_l *= alpha;
            m_run = m_new;
#pragma unroll
            for (int db = 0; db < S::kBlocks; ++db) acc[db] *= alpha;
            probabilities(m_new);
        }
        l_run += lsum;
        seg_l += lsum;
        // ---- O^T += V^T P^T
        if constexpr (S::kF32) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float* vr = reinterpret_cast<const float*>(v_lds + (4 * lg + r) * S::kVRow) + li;
#pragma unroll
                for (int db = 0; db < S::kBlocks; ++db) acc[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[16 * db], pv[r], acc[db], 0, 0, 0);
            }
        } else {
            uint4 pp[S::kPParts];
#pragma unroll
            for (int n = 0; n < S::kPParts; ++n) pp[n] = split_part<DT>(reinterpret_cast<float (&)[8]>(pv), DT == CF_F16 ? 2048.f : 1.f);
            const unsigned char* vb = v_lds + (4 * lg + (li >> 2)) * S::kVRow + 8 * (li & 3);
#pragma unroll
            for (int db = 0; db < S::kBlocks; ++db) {
                const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)(vb + 32 * db));
                const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)(vb + 32 * db + 16 * S::kVRow));
                const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
                const uint4 va = make_uint4(l2.x, l2.y, h2.x, h2.y);
                if constexpr (DT == CF_F16) {                // the scaled parts' sum joins the first's; three chains (one: up to 6 % slower)
                    const f32x4 none = f32x4{0.f, 0.f, 0.f, 0.f};
                    const f32x4 t = Mma<CF_F16>::run(va, pp[1], none), u = Mma<CF_F16>::run(va, pp[2], none);
                    acc[db] = Mma<CF_F16>::run(va, pp[0], acc[db]) + (t + u * 0x1p-11f) * 0x1p-11f;
                } else {
#pragma unroll
                    for (int n = S::kPParts - 1; n >= 0; --n) acc[db] = Mma<CF_BF16>::run(va, pp[n], acc[db]);
                }
            }
        }
    };

    char* ws = static_cast<char*>(a.workspace);
    const int rows = 16 * RB;
    // slot statistics: [query, kv head][slot][row], for the rows there are and not for those a block is padded to
    const int rows_kv = group * a.max_tq;
    float2* massml = reinterpret_cast<float2*>(ws + p.off_massml) + ((int64_t)b * a.n_kv_heads + hkv) * p.slots * rows_kv + row_base;
    auto emit = [&](int slot) __attribute__((always_inline)) {                              // (reference, sum) of the segment per row
        float tot = seg_l + __shfl_xor(seg_l, 16);
        tot += __shfl_xor(tot, 32);
        if (lg == 0 && row_ok) massml[(int64_t)slot * rows_kv + wave * 16 + li] = make_float2(m_run, tot);
    };

    // Row rr of the wavefront's block over all the tokens of the workgroup, as the row-by-row kernel goes over them: only what the row
    // sees is read, keys are turned and products summed in fp32.  Same records as emit.
    auto redo_row = [&](int rr, float (&o)[4], float& m, float& l) {
        using E = Elem<DT>;
        using T = typename E::type;
        // (the kernel's first argument read anew: kept in registers for this, its fields would crowd those of the main loop)
        uint64_t kernarg = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
        uint32_t lo = (uint32_t)kernarg, hi = (uint32_t)(kernarg >> 32);
        asm volatile("" : "+v"(lo), "+v"(hi));
        kernarg = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)hi) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
        const auto* ka = reinterpret_cast<const __attribute__((address_space(4))) AttnArgs*>(kernarg);
        const int half = d >> 1, row = row_base + wave * 16 + rr;
        const int head = (int)div_exact((unsigned)row, (unsigned)tq), t = row - head * tq;
        const T* qp = static_cast<const T*>(ka->q) + (((int64_t)qh.q0 + t) * ka->n_q_heads + hkv * group + head) * d;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = 0.f;
        auto lane_of = [](float x, int from) { return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), from)); };
        m = -INFINITY;
        l = 0.f;
        for (int g = 0; g < kGroups; ++g) {
            const int sub = split * kGroups + g;
            TileWalk<S::kTile> from(split_begin(total, nsub, sub), split_begin(total, nsub, sub + 1));
            int seg = -1;
            float sum = 0.f;
            float2 cs_lo = {}, cs_hi = {};                   // slices lane, lane + 64
            for (;;) {
                const Tile c = reg_table ? from.next(rtbl, lane) : from.next(tbl, lane);
                if (c.ntok == 0 || c.seg != seg) {
                    if (seg >= 0 && lane == 0) massml[(int64_t)(seg + sub) * rows_kv + wave * 16 + rr] = make_float2(m, sum);
                    if (c.ntok == 0) break;
                    seg = c.seg;
                    sum = 0.f;
                    cs_lo = rope_cos_sin(c.delta, freq.rev[min(lane, half - 1)]);
                    if (half > kWave) cs_hi = rope_cos_sin(c.delta, freq.rev[min(lane + kWave, half - 1)]);
                }
                const int vis = c.self ? min(c.ntok, t + 1 - c.tok0) : c.ntok;
                if (vis <= 0) continue;
                const int64_t ts = c.self ? (int64_t)ka->n_kv_heads * d : ka->store_ts;
                const int64_t base = (from.c_tok + c.tok0) * ts + (int64_t)hkv * (c.self ? d : ka->store_hs);
                const T* kp = static_cast<const T*>(c.self ? ka->k_self : ka->k_store) + base + min(lane, vis - 1) * ts;
                const T* vp = static_cast<const T*>(c.self ? ka->v_self : ka->v_store) + base;
                float sc = 0.f;
                for (int n = 0; n < half; ++n) {             // (every lane, past the visible tokens too: lane reads are not for branches)
                    const int c0 = ka->pairing == CF_ROPE_HALF ? n : 2 * n, c1 = ka->pairing == CF_ROPE_HALF ? n + half : 2 * n + 1;
                    float x = E::load(kp + c0), y = E::load(kp + c1);
                    if (c.delta != 0) {
                        const float2 w = n < kWave ? cs_lo : cs_hi;
                        const float2 u = make_float2(lane_of(w.x, n & (kWave - 1)), lane_of(w.y, n & (kWave - 1)));
                        const float nx = x * u.x - y * u.y;
                        y = x * u.y + y * u.x;
                        x = nx;
                    }
                    sc += E::load(qp + c0) * x + E::load(qp + c1) * y;
                }
                sc = lane < vis ? sc * ka->scale_log2e : -INFINITY;
                const float m_new = fmaxf(m, wave_max(sc)), m_ref = m_new == -INFINITY ? 0.f : m_new;
                const float alpha = exp2f(m - m_ref), pr = lane < vis ? exp2f(sc - m_ref) : 0.f;
                const float add = wave_sum(pr);
                l = l * alpha + add;
                sum = sum * alpha + add;
                m = m_new;
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] *= alpha;
                for (int j = 0; j < vis; ++j) {
                    const float pj = lane_of(pr, j);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (lane + kWave * i < d) o[i] += pj * E::load(vp + j * ts + lane + kWave * i);
                }
            }
        }
    };

    Tile nxt;
    fetch(nxt, regs);
    int cs_slot = 0, cur_seg = -1;
    if (nxt.ntok > 0 && nxt.delta != 0) make_angles(nxt, 0);
    for (int it = 0; it < most_tiles; ++it) {
        const Tile cd = nxt;
        const int cd_slot = cs_slot;
        unsigned char* k_lds = bufs[grp][kBufs == 2 ? it & 1 : 0];
        unsigned char* v_lds = k_lds + S::kTile * S::kKRow;
        if (cd.ntok > 0) {
#pragma unroll
            for (int i = 0; i < kItems; ++i) {
                *reinterpret_cast<u32x4*>(k_lds + (sr + i * kSweep) * S::kKRow + 16 * sc) = regs.k[i];
                *reinterpret_cast<u32x4*>(v_lds + (sr + i * kSweep) * S::kVRow + 16 * sc) = regs.v[i];
            }
        }
        fetch(nxt, regs);
        // angles go round three slots: a wavefront may still read this tile's while another makes those of the tile after next
        if (nxt.ntok > 0 && nxt.seg != cd.seg && nxt.delta != 0) {
            cs_slot = cs_slot == 2 ? 0 : cs_slot + 1;
            make_angles(nxt, cs_slot);
        }
        __syncthreads();
        if (cd.ntok > 0 && has_rows) {
            if (cd.seg != cur_seg) {
                if (cur_seg >= 0) emit(cur_seg + ss);
                cur_seg = cd.seg;
                seg_l = 0.f;
                turn_query(cd, cd_slot);
            }
            tile_pass(cd, k_lds, v_lds);
        }
        if constexpr (kBufs == 1) __syncthreads();
    }
    if (cur_seg >= 0) emit(cur_seg + ss);
    float l_row = l_run + __shfl_xor(l_run, 16);
    l_row += __shfl_xor(l_row, 32);

    // ---- the groups' results (same rows, other tokens) meet in the first group, through the tile buffers
    if constexpr (kGroups > 1) {
        static_assert((kGroups - 1) * RB * S::kBlocks * kWave * 16 <= kGroups * kBufs * S::kBuf, "the exchange fits the tile buffers");
        f32x4* red = reinterpret_cast<f32x4*>(&bufs[0][0][0]);
        __syncthreads();
        if (grp > 0) {
#pragma unroll
            for (int db = 0; db < S::kBlocks; ++db) red[(((grp - 1) * RB + wave) * S::kBlocks + db) * kWave + lane] = acc[db];
        }
        if (lg == 0) ml_lds[grp][wave * 16 + li] = make_float2(m_run, l_row);
        __syncthreads();
        if (grp == 0) {
            float m = m_run;
#pragma unroll
            for (int g = 1; g < kGroups; ++g) m = fmaxf(m, ml_lds[g][wave * 16 + li].x);
            const float ms = m == -INFINITY ? 0.f : m;
            const float f0 = __builtin_amdgcn_exp2f(m_run - ms);
            l_row *= f0;
#pragma unroll
            for (int db = 0; db < S::kBlocks; ++db) acc[db] *= f0;
#pragma unroll
            for (int g = 1; g < kGroups; ++g) {
                const float2 o = ml_lds[g][wave * 16 + li];
                const float f = __builtin_amdgcn_exp2f(o.x - ms);
                l_row += o.y * f;
#pragma unroll
                for (int db = 0; db < S::kBlocks; ++db) acc[db] += red[(((g - 1) * RB + wave) * S::kBlocks + db) * kWave + lane] * f;
            }
            m_run = m;
        }
    }
    // ---- rows that did not stay finite: a tile's product multiplies tokens a row does not see by zero, and the parts of a number
    // do not add up to infinities, so these rows go over the workgroup's tokens once more, one by one
    if (grp == 0 && has_rows) {
        float zero = l_row * 0.f;
#pragma unroll
        for (int db = 0; db < S::kBlocks; ++db)
#pragma unroll
            for (int e = 0; e < 4; ++e) zero = fmaf(acc[db][e], 0.f, zero);
        const unsigned long long lost = __ballot(row_ok && !(zero == 0.f));
        if (__builtin_expect(lost != 0, 0)) for (unsigned left = (unsigned)(lost | lost >> 16 | lost >> 32 | lost >> 48) & 0xffffu; left != 0; left &= left - 1) {
            const int rr = __builtin_ctz(left);
            float o[4], m, l;                                // channels lane, lane + 64, ...
            redo_row(rr, o, m, l);
            if (li == rr) { m_run = m; l_row = l; }
#pragma unroll
            for (int db = 0; db < S::kBlocks; ++db)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = __shfl(o[db / 4], (16 * db + 4 * lg + e) & (kWave - 1));
                    if (li == rr) acc[db][e] = x;
                }
        }
    }
    const float inv = l_row > 0.f ? 1.f / l_row : 0.f;
    if (grp == 0 && has_rows) {
        if (!p.direct_out) {
            float2* ml = reinterpret_cast<float2*>(ws + p.off_ml) + ((int64_t)unit * p.nsplit + split) * rows;
            f32x4* opart = reinterpret_cast<f32x4*>(ws + p.off_opart) + (((int64_t)unit * p.nsplit + split) * RB + wave) * S::kBlocks * kWave + lane;
            if (lg == 0) ml[wave * 16 + li] = make_float2(m_run, l_row);
#pragma unroll
            for (int db = 0; db < S::kBlocks; ++db)
                if (16 * db < d) opart[db * kWave] = acc[db] * inv;
        } else if (row_ok) {
            using E = Elem<DT>;
            typename E::type* op = static_cast<typename E::type*>(a.out) + (((int64_t)qh.q0 + t_row) * a.n_q_heads + hkv * group + gi) * d + 4 * lg;
#pragma unroll
            for (int db = 0; db < S::kBlocks; ++db)
                if (16 * db < d) {
                    const f32x4 o = acc[db] * inv;
                    if constexpr (S::kF32) {
                        *reinterpret_cast<f32x4*>(op + 16 * db) = o;
                    } else {
                        *reinterpret_cast<uint2*>(op + 16 * db) = make_uint2(Mma<DT>::pack(o[0], o[1]), Mma<DT>::pack(o[2], o[3]));
                    }
                }
        }
    }
    // ---- one split: the rows' statistics are final, so the slots are reduced here (else by the merge kernel)
    if (p.direct_out && a.mass != nullptr) {
        __syncthreads();                                     // publishes the slots (and everybody has read ml_lds)
        if (grp == 0 && lg == 0) ml_lds[0][wave * 16 + li] = make_float2(m_run, row_ok ? l_row : 0.f);
        __syncthreads();
        double* part = reinterpret_cast<double*>(ws + p.off_masspart) + (int64_t)unit * p.slots;
        const float2 st = lane < rows ? ml_lds[0][lane] : make_float2(0.f, 0.f);
        for (int k = wave_all; k < p.slots; k += kWaves) {
            const float2 v = lane < row_limit - row_base ? massml[(int64_t)k * rows_kv + lane] : make_float2(0.f, 0.f);
            const double c = wave_sum_f64(slot_share(v, st));
            if (lane == 0) part[k] = c;
        }
    }
}

// Merges the splits' partial rows and writes the output rows; with MASS reduces the slots to the unit's partial masses.  One wavefront per
// (row block, 16 channels) of a unit; grid (unit of the query, sets of four wavefronts, query), so that a unit's workgroups share an XCD where
// eight divides the units.  Bound by its two dependent round trips (arguments, one batch of loads): each wavefront works its rows' statistics
// out for itself and shares nothing.  NS: splits whose statistics are held in registers.  blocks: log2 of the channel blocks.
// With the statistics worked out by one thread per row out of LDS behind two barriers: 32 units x 16 splits x 48 rows 8.3 -> 5.7 us.
template <int DT, int NS, bool MASS>
__global__ __launch_bounds__(kThreads) void plain_combine_kernel(AttnArgs a, Plan p, int blocks) {
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int li = lane & 15, lg = lane >> 4;
    const int b = blockIdx.z, unit = b * p.units_per_b + (int)blockIdx.x;
    const int hkv = p.n_rg == 1 ? (int)blockIdx.x : (int)div_exact(blockIdx.x, (unsigned)p.n_rg);
    const int rg = (int)blockIdx.x - hkv * p.n_rg;
    const int rows = p.rows_wg, rbs = rows / 16;
    const int item = blockIdx.y * kWaves + wave;             // row block, channel block (at least four channel blocks: no wavefront is left over)
    const int rb = item >> blocks, db = item - (rb << blocks);
    char* ws = static_cast<char*>(a.workspace);
    // with MASS lane r holds row r of the unit, which the slots are reduced over, else the row of the lane's partial outputs
    const int row = MASS ? min(lane, rows - 1) : rb * 16 + li;
    const float2* ml = reinterpret_cast<const float2*>(ws + p.off_ml) + (int64_t)unit * p.nsplit * rows + row;
    const f32x4* src = reinterpret_cast<const f32x4*>(ws + p.off_opart) + ((((int64_t)unit * p.nsplit * rbs + rb) << blocks) + db) * kWave + lane;
    const int64_t stride = (int64_t)(rbs << blocks) * kWave;
    const int q0 = a.q_off[b], q1 = a.q_off[b + 1];
    const int row_base = rg * p.blocks_rg * 16;
    const int rows_kv = p.group * a.max_tq;
    const float2* massml = reinterpret_cast<const float2*>(ws + p.off_massml) + ((int64_t)b * a.n_kv_heads + hkv) * p.slots * rows_kv + row_base +
                           min(lane, rows_kv - row_base - 1);
    const int k_step = (int)gridDim.y * kWaves;
    // one batch of unconditional loads: rows without a query are read (what an earlier call left there) and dropped
    float2 st[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) st[s] = ml[(int64_t)min(s, p.nsplit - 1) * rows];
    constexpr int kPre = NS == 16 ? 16 : 8;
    f32x4 pre[kPre];
#pragma unroll
    for (int s = 0; s < kPre; ++s) pre[s] = src[min(s, p.nsplit - 1) * stride];
    constexpr int kSv = 4;
    float2 sv[kSv];
    if constexpr (MASS) {
#pragma unroll
        for (int j = 0; j < kSv; ++j) sv[j] = massml[(int64_t)min(item + j * k_step, p.slots - 1) * rows_kv];
    }
    __builtin_amdgcn_sched_barrier(0);
    const int tq = min(q1 - q0, a.max_tq);
    const int rows_here = min(p.blocks_rg * 16, p.group * tq - row_base);
    float m = -INFINITY;
#pragma unroll
    for (int s = 0; s < NS; ++s) m = fmaxf(m, st[s].x);
    m = m == -INFINITY ? 0.f : m;
    float z = 0.f, weight[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        weight[s] = s < p.nsplit ? st[s].y * exp2f(st[s].x - m) : 0.f;
        z += weight[s];
    }
    auto of_block = [&](float x) { return MASS ? __shfl(x, (rb * 16 + li) & (kWave - 1)) : x; };
    f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
    int n_splits = p.nsplit;
#ifdef __OPTIMIZE__
    asm volatile("" : "+s"(n_splits));                       // (the comparisons above are not kept for those below: 32 pairs of scalar registers)
#endif
#pragma unroll
    for (int s0 = 0; s0 < NS; s0 += kPre) {
        if (s0 >= n_splits) break;
        if (s0 > 0) {
#pragma unroll
            for (int i = 0; i < kPre; ++i) pre[i] = src[min(s0 + i, p.nsplit - 1) * stride];
        }
        float w[kPre];
#pragma unroll
        for (int i = 0; i < kPre; ++i) w[i] = of_block(weight[s0 + i]);
#pragma unroll
        for (int i = 0; i < kPre; ++i)
            if (s0 + i < n_splits) o += pre[i] * w[i];
    }
    const float z_row = of_block(z);
    o *= z_row > 0.f ? 1.f / z_row : 0.f;
    const int lrow = rb * 16 + li;
    if (lrow < rows_here && 16 * db < a.head_dim) {
        const int m2 = row_base + lrow;
        const int gi = (int)div_exact((unsigned)m2, (unsigned)tq), t = m2 - gi * tq;
        using E = Elem<DT>;
        typename E::type* op = static_cast<typename E::type*>(a.out) +
                               (((int64_t)q0 + t) * a.n_q_heads + hkv * p.group + gi) * a.head_dim + 16 * db + 4 * lg;
        if constexpr (DT == CF_F32) {
            *reinterpret_cast<f32x4*>(op) = o;
        } else {
            *reinterpret_cast<uint2*>(op) = make_uint2(Mma<DT>::pack(o[0], o[1]), Mma<DT>::pack(o[2], o[3]));
        }
    }
    if constexpr (MASS) {
        double* part = reinterpret_cast<double*>(ws + p.off_masspart) + (int64_t)unit * p.slots;
        const float2 stat = make_float2(m, lane < rows_here ? z : 0.f);      // (slot_share: a row sum of 0 is no such row)
        auto reduce = [&](int k, float2 v) {
            const double c = wave_sum_f64(slot_share(v, stat));
            if (lane == 0 && k < p.slots) part[k] = c;
        };
#pragma unroll
        for (int j = 0; j < kSv; ++j)
            if (item + j * k_step < p.slots) reduce(item + j * k_step, sv[j]);
        for (int k = item + kSv * k_step; k < p.slots; k += k_step) reduce(k, massml[(int64_t)k * rows_kv]);
    }
}

int padded_dim(int d) { return d <= 64 ? 64 : d <= 128 ? 128 : 256; }

// most: the plan that the bytes reported are those of, which a call's own never takes more than.
Plan make_plain_plan(const cf_layer_desc& d, int batch, int max_tq, int seg_stride, int64_t max_kv_tokens, bool most = false) {
    Plan p = {};
    const int dp = padded_dim(d.head_dim);
    p.group = d.n_q_heads / d.n_kv_heads;
    p.row_blocks = (p.group * max_tq + 15) / 16;
    // row blocks a workgroup has room for (the widest heads' registers and tiles leave no room for four groups)
    const int rb = p.row_blocks == 1 && dp < 256 ? 1 : p.row_blocks <= 2 ? 2 : 4;
    p.n_rg = (p.row_blocks + rb - 1) / rb;
    p.blocks_rg = (p.row_blocks + p.n_rg - 1) / p.n_rg;
    p.nrb = 1;
    p.rows_wg = 16 * rb;
    p.groups = kWaves / rb;
    p.tile = d.dtype == CF_F32 ? 16 : 32;
    p.units_per_b = d.n_kv_heads * p.n_rg;
    p.units = batch * p.units_per_b;
    // Enough splits to fill the CUs.  A group keeps at least two tiles, and a
    // list that gives every group at most four is not split at all: the merge kernel would cost more than it saves.
    const int64_t est_tiles = max_kv_tokens / p.tile + seg_stride / 2;
    int64_t ns = 256 * plain_per_cu(d.dtype == CF_F32, dp, rb) / p.units;
    const int64_t cap = est_tiles / (2 * p.groups);
    if (ns > cap) ns = cap;
    if (ns * p.groups > kMaxSplit) ns = kMaxSplit / p.groups;
    // More than eight splits of fewer than four tiles a group: the merge costs more than two workgroups to a CU save, where eight fill the CUs
    // once.  us with up to sixteen and with eight, tiles in brackets: bf16, 5 documents x 32 heads (2.1) 23.0 and 20.8, 10 (3.5) 27.0 and 26.7,
    // 16 queries x 2 heads (2.1) 22.3 and 21.0; fp32, 10 documents x 32 heads (3.2) 25.7 and 24.6, 7 (2.8) 30.0 and 28.9; but (5.6) 36.8 and
    // 39.7, (12.7) 39.3 and 46.5, bf16 (6.8) 26.7 and 28.3.  fp16, whose tiles take longer: (2.3) 27.7 and 28.1, (3.5) 28.4 and 29.6.
    // Not in the bytes reported: smaller batches and longer lists are split further than that, and a workspace serves them as far as it did
    // without this rule.
    if (!most && d.dtype != CF_F16 && ns > 8 && p.units >= 32 && est_tiles < 4 * p.groups * ns) ns = 8;
    if (ns < 1 || est_tiles <= 4 * p.groups) ns = 1;
    p.nsplit = (int)ns;
    p.direct_out = p.nsplit == 1;
    p.slots = seg_stride + p.nsplit * p.groups;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) & ~(size_t)255; return o; };
    p.off_ml = take(p.direct_out ? 0 : (size_t)p.units * p.nsplit * p.rows_wg * sizeof(float2));
    p.off_opart = take(p.direct_out ? 0 : (size_t)p.units * p.nsplit * p.rows_wg * dp * sizeof(float));
    p.off_massml = take((size_t)batch * d.n_kv_heads * p.slots * p.group * max_tq * sizeof(float2));
    p.masspart_bytes = ((size_t)p.units * p.slots * sizeof(double) + 255) & ~(size_t)255;
    p.off_masspart = take(p.masspart_bytes);
    p.total = off;
    return p;
}

template <int DT>
void launch_plain(const AttnArgs& a, const RopeFreq& f, const Plan& p, hipStream_t s) {
    const dim3 grid((unsigned)p.nsplit, (unsigned)p.units_per_b, (unsigned)a.batch), block(kThreads);
#define CF_PLAIN(DP, RB) hipLaunchKernelGGL((attn_plain_kernel<DT, DP, RB>), grid, block, 0, s, a, f, p)
#define CF_PLAIN_D(DP)                                    \
    if (p.rows_wg == 16) CF_PLAIN(DP, 1);                 \
    else if (p.rows_wg == 32) CF_PLAIN(DP, 2);            \
    else CF_PLAIN(DP, 4)
    switch (padded_dim(a.head_dim)) {
        case 64: CF_PLAIN_D(64); break;
        case 128: CF_PLAIN_D(128); break;
        default:
            if (p.rows_wg == 32) CF_PLAIN(256, 2);
            else CF_PLAIN(256, 4);
            break;
    }
#undef CF_PLAIN_D
#undef CF_PLAIN
    if (p.direct_out) return;
    const int blocks = padded_dim(a.head_dim) / 16;
    const dim3 cgrid((unsigned)p.units_per_b, (unsigned)(p.rows_wg / 16 * blocks / kWaves), (unsigned)a.batch);
#define CF_COMBINE(NS)                                                                                                          \
    if (a.mass != nullptr) hipLaunchKernelGGL((plain_combine_kernel<DT, NS, true>), cgrid, block, 0, s, a, p, __builtin_ctz(blocks)); \
    else hipLaunchKernelGGL((plain_combine_kernel<DT, NS, false>), cgrid, block, 0, s, a, p, __builtin_ctz(blocks))
    if (p.nsplit <= 8) { CF_COMBINE(8); }
    else if (p.nsplit <= 16) { CF_COMBINE(16); }
    else { CF_COMBINE(kMaxSplit); }
#undef CF_COMBINE
}

}  // namespace

// Tables past kMaxSegs entries, grids past the hardware's and counts past the plan's 32 bits stay with the row-by-row kernel, and so
// do many queries of a row or two over a few tokens: a workgroup takes the 10 us of its round trips (23 at 256 channels) whatever
// it holds, a CU has one or two of them, and a wavefront per row is through such a row in a fraction of that.  A row there costs about
// as much as 45 tokens.  256 queries x 32 heads, row by row against this kernel: fp32, d = 64, 1 row over 21 tokens 64 and 157 us, over 61
// 102 and 161, over 201 322 and 267; 3 rows over 23 162 and 159; bf16, d = 128 (one workgroup per CU), 1 row over 61 161 and 367, over
// 201 500 and 466; fp16, d = 256, 1 row over 21 163 and 740.  64 queries x 32 heads: fp32 25 and 45, 46 and 49, 101 and 71; 16 x 32: 25
// and 18, 31 and 17.
bool plain_path_supported(const cf_layer_desc* d, int32_t batch, int32_t max_tq, int32_t seg_stride, int64_t max_kv_tokens) {
    const int64_t rows = (int64_t)(d->n_q_heads / d->n_kv_heads) * max_tq, units_per_b = d->n_kv_heads * ((rows + 63) / 64 + 1);
    const int64_t few = plain_per_cu(d->dtype == CF_F32, padded_dim(d->head_dim), 1) == 1 ? 160 : 110;
    if ((int64_t)batch * d->n_kv_heads >= 2048 && rows <= 3 && max_kv_tokens <= few && rows * (max_kv_tokens + 45) <= few) return false;
    return seg_stride <= kMaxSegs && batch <= 65535 && rows < (1 << 20) && units_per_b <= 65535 && batch * units_per_b <= 0x7fffffff;
}

size_t plain_workspace_bytes(const cf_layer_desc* d, int32_t batch, int32_t max_tq, int32_t seg_stride, int64_t max_kv_tokens) {
    return make_plain_plan(*d, batch, max_tq, seg_stride, max_kv_tokens, true).total;
}

size_t plain_call_bytes(const cf_layer_desc* d, int32_t batch, int32_t max_tq, int32_t seg_stride, int64_t max_kv_tokens) {
    return make_plain_plan(*d, batch, max_tq, seg_stride, max_kv_tokens).total;
}

cf_status launch_attention_plain(const cf_layer_desc* d, AttnArgs a, const RopeFreq& f, hipStream_t s, const cf_prune_step* prune) {
    const Plan p = make_plain_plan(*d, a.batch, a.max_tq, a.seg_stride, a.max_kv_tokens);
    a.n_pending = 0;                                         // scores are never deferred here
    a.defer = 0;
    switch (a.dtype) {
        case CF_F32: launch_plain<CF_F32>(a, f, p, s); break;
        case CF_BF16: launch_plain<CF_BF16>(a, f, p, s); break;
        default: launch_plain<CF_F16>(a, f, p, s); break;
    }
    CF_HIP(hipGetLastError());
    if (prune && epilogue_fits_f64(p, prune)) {
        launch_epilogue_f64(a, p, prune, s);
    } else if (a.mass != nullptr) {
        launch_mass_f64(a, p, s);
        CF_HIP(hipGetLastError());
        if (prune) return launch_prune_step(a, prune, s);
    }
    CF_HIP(hipGetLastError());
    return CF_OK;
}

}  // namespace cf
