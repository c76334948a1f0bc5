// Cache Re-Positioning, materialised (Sec. 2.3, Eq. 5): every key of every listed segment is
// rotated from the position it was cached at to its new position.  Pure streaming kernel:
// 16-byte loads and stores, one read and one write of K, bound by HBM bandwidth.
#include "cf_common.h"

namespace cf {
namespace {

constexpr int kThreads = 256;
constexpr int kPanelItems = 1 << 20;   // items of a segment that are numbered together: div_exact stays on its short path

// Eight consecutive elements as they lie in memory, and as floats.  Compiler vectors and not HIP's uint4 / float4:
// arrays of those classes that are only copied stayed in memory (LDS or scratch) instead of registers.
using U4 = uint32_t __attribute__((ext_vector_type(4)));
using F4 = float __attribute__((ext_vector_type(4)));
template <int DT> struct Chunk8 {
    U4 r;
    __device__ __forceinline__ void load(const void* base, int64_t idx) {
        r = *reinterpret_cast<const U4*>(static_cast<const uint16_t*>(base) + idx);
    }
    template <bool STREAM> __device__ __forceinline__ void store(void* base, int64_t idx) const {
        U4* p = reinterpret_cast<U4*>(static_cast<uint16_t*>(base) + idx);
        if constexpr (STREAM) __builtin_nontemporal_store(r, p);
        else *p = r;
    }
    __device__ __forceinline__ void to_float(float (&v)[8]) const {
        const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (DT == CF_BF16) {
                v[2 * i] = bf16_bits_to_float(w[i] & 0xffffu);
                v[2 * i + 1] = bf16_bits_to_float(w[i] >> 16);
            } else {
                v[2 * i] = f16_bits_to_float(w[i] & 0xffffu);
                v[2 * i + 1] = f16_bits_to_float(w[i] >> 16);
            }
        }
    }
    __device__ __forceinline__ void from_float(const float (&v)[8]) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (DT == CF_BF16)
                w[i] = float_to_bf16_bits(v[2 * i]) | (float_to_bf16_bits(v[2 * i + 1]) << 16);
            else
                w[i] = float_to_f16_bits(v[2 * i]) | (float_to_f16_bits(v[2 * i + 1]) << 16);
        }
        r = U4{w[0], w[1], w[2], w[3]};
    }
};
template <> struct Chunk8<CF_F32> {
    F4 a, b;
    __device__ __forceinline__ void load(const void* base, int64_t idx) {
        const F4* p = reinterpret_cast<const F4*>(static_cast<const float*>(base) + idx);
        a = p[0];
        b = p[1];
    }
    template <bool STREAM> __device__ __forceinline__ void store(void* base, int64_t idx) const {
        F4* p = reinterpret_cast<F4*>(static_cast<float*>(base) + idx);
        p[0] = a;
        p[1] = b;
    }
    __device__ __forceinline__ void to_float(float (&v)[8]) const {
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
    __device__ __forceinline__ void from_float(const float (&v)[8]) {
        a = F4{v[0], v[1], v[2], v[3]};
        b = F4{v[4], v[5], v[6], v[7]};
    }
};

// A work item is 8 pairs of one (token, kv head): under half-split pairing the 8 first elements [8j, 8j+8) and
// their partners [d/2+8j, ...); under interleaved pairing 16 consecutive elements.  Items of a run of tokens are
// numbered along the memory of the layout - token rows of one head after another where a head's tokens lie together
// (by_head), else heads within a token - so that a block's items are one contiguous piece of a few KB and not
// 256-byte rows a head stride apart.
struct Item {
    int tok, head, j;
};
__device__ __forceinline__ Item locate(int it, int items_per_head, int heads, int ntok, bool by_head) {
    const int row = (int)div_exact((unsigned)it, (unsigned)items_per_head);
    const int inner = by_head ? ntok : heads;
    const int outer = (int)div_exact((unsigned)row, (unsigned)inner);
    const int rest = row - outer * inner;
    return {by_head ? rest : outer, by_head ? outer : rest, it - row * items_per_head};
}

// first and second 16-bit-wide (or fp32) chunk of an item within its row
template <int PAIRING> __device__ __forceinline__ int first_of(int j) { return PAIRING == CF_ROPE_HALF ? 8 * j : 16 * j; }
template <int PAIRING> __device__ __forceinline__ int second_of(int j, int half) {
    return PAIRING == CF_ROPE_HALF ? half + 8 * j : 16 * j + 8;
}

template <int DT, int PAIRING>
__device__ __forceinline__ void rotate(Chunk8<DT>& c0, Chunk8<DT>& c1, const float2* cs, int j) {
    float a[8], b[8];
    c0.to_float(a);
    c1.to_float(b);
    if (PAIRING == CF_ROPE_HALF) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float2 w = cs[8 * j + e];
            const float na = a[e] * w.x - b[e] * w.y;
            const float nb = a[e] * w.y + b[e] * w.x;
            a[e] = na;
            b[e] = nb;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float2 w0 = cs[8 * j + e];
            const float x0 = a[2 * e] * w0.x - a[2 * e + 1] * w0.y;
            const float y0 = a[2 * e] * w0.y + a[2 * e + 1] * w0.x;
            a[2 * e] = x0;
            a[2 * e + 1] = y0;
            const float2 w1 = cs[8 * j + 4 + e];
            const float x1 = b[2 * e] * w1.x - b[2 * e + 1] * w1.y;
            const float y1 = b[2 * e] * w1.y + b[2 * e + 1] * w1.x;
            b[2 * e] = x1;
            b[2 * e + 1] = y1;
        }
    }
    c0.from_float(a);
    c1.from_float(b);
}

// 16-bit types are written past the caches.  30 documents x 160 tokens of 32 heads, bf16: assembly 36.2 -> 30.0 us (5.2 TB/s read and written, the
// rate of a large copy); 2 x 18 documents of 66-121 tokens, 32 heads, token-major: 28.7 -> 21.1; interleaved pairs 7.3 -> 6.6 and 11.1 -> 10.0;
// re-positioning the same within the noise.  What reads the cache next finds it in memory: the assembly of 30 documents and a decode step over
// them right behind it 55.8 and 56.2 us, of 5 documents 21.1 and 20.5.  Not fp32, whose store instructions leave
// every other 16 bytes to the next one (re-positioning 84 documents of 53 tokens, 4 heads: 6.8 and 8.4 us).  Loads past the caches:
// re-positioning 13.4 -> 15.3, assembly the same.
template <int DT> constexpr bool kStream = DT != CF_F32;

// Where a block works in a segment of `len` tokens: panels of whole tokens, in each the block's chunk of U * kThreads
// items, then those a grid further on.  Every block of a segment visits the same panels.
template <int U> struct Walk {
    int len, panel, per_tok, tok0, at;
    __device__ Walk(int len_, int per_tok_) : len(len_), panel(max(1, kPanelItems / per_tok_)), per_tok(per_tok_), tok0(0) {
        at = blockIdx.y * (U * kThreads);
        settle();
    }
    __device__ int ntok() const { return min(panel, len - tok0); }
    __device__ int n_items() const { return ntok() * per_tok; }
    __device__ bool more() const { return tok0 < len; }
    __device__ void next() {
        at += gridDim.y * (U * kThreads);
        settle();
    }
    __device__ void settle() {
        while (more() && at >= n_items()) {
            tok0 += ntok();
            at = blockIdx.y * (U * kThreads);
        }
    }
};

// grid = (n_seg, pieces of a segment); block = 256 threads, an item each.  Bound by HBM, one read and one write of K;
// a block's loads are requested before the cos/sin table is worked out, which hides behind them.  One item per thread:
// two or four were slower at every size (30 documents x 160 tokens of 32 heads, bf16: 13.8 us against 14.5 and 14.3, 5.7 TB/s
// read and written; 16 fp32 documents of 50-79 tokens 8.8 against 9.5 and 10.0).
template <int DT, int PAIRING>
__global__ __launch_bounds__(kThreads) void reposition_kernel(
    const void* k_in, void* k_out, const cf_segment* __restrict__ segs,
    int64_t n_store_tokens, int n_kv_heads, int head_dim, int64_t tok_stride, int64_t head_stride, RopeFreq freq,
    int32_t* dev_flag, int max_positions) {
    __shared__ float2 cs[kMaxHalf];
    const cf_segment seg = segs[blockIdx.x];
    const int half = head_dim >> 1;
    if (seg.len < 0 || seg.tok_offset < 0 || seg.tok_offset + seg.len > n_store_tokens) {
        if (threadIdx.x == 0 && blockIdx.y == 0) raise_flag(dev_flag, CF_FLAG_BAD_SEGMENT);
        return;
    }
    if (!positions_ok(seg.stored_start, seg.len, max_positions) || !positions_ok(seg.new_start, seg.len, max_positions)) {
        if (threadIdx.x == 0 && blockIdx.y == 0) raise_flag(dev_flag, CF_FLAG_POS_RANGE);
        return;
    }
    const int items_per_head = half / 8;                 // head_dim % 16 == 0 checked on the host
    const bool by_head = head_stride > tok_stride;
    Walk<1> walk(seg.len, n_kv_heads * items_per_head);
    if (!walk.more()) return;                            // the whole block
    const int delta = seg.new_start - seg.stored_start;
    bool table = false;
    for (; walk.more(); walk.next()) {
        const int n_items = walk.n_items(), it = walk.at + (int)threadIdx.x;
        // an item past the end reads the last one again and stores nothing
        const Item i = locate(min(it, n_items - 1), items_per_head, n_kv_heads, walk.ntok(), by_head);
        const int64_t base = (seg.tok_offset + walk.tok0 + i.tok) * tok_stride + (int64_t)i.head * head_stride;
        const int64_t o0 = base + first_of<PAIRING>(i.j), o1 = base + second_of<PAIRING>(i.j, half);
        Chunk8<DT> a, b;
        a.load(k_in, o0);
        b.load(k_in, o1);
        if (!table) {
            for (int m = threadIdx.x; m < half; m += kThreads) cs[m] = rope_cos_sin(delta, freq.rev[m]);
            __syncthreads();
            table = true;
        }
        if (it >= n_items) continue;
        rotate<DT, PAIRING>(a, b, cs, i.j);
        a.template store<kStream<DT>>(k_out, o0);
        b.template store<kStream<DT>>(k_out, o1);
    }
}

// Pieces of a segment: all of them for the stated longest length, as long as the launch stays within `most` blocks; the blocks there
// are walk the rest.  The stated length may be far above the real ones, and a block that finds nothing to do still costs its start.
unsigned pieces(int64_t n_seg, int32_t max_seg_len, int per_tok, int unroll, int64_t most) {
    const int64_t n = ((int64_t)max_seg_len * per_tok + unroll * kThreads - 1) / (unroll * kThreads);
    const int64_t each = most / n_seg > 1 ? most / n_seg : 1;
    return (unsigned)(n > each ? each : n);
}
// Four times what fills the chip.  At a fitting stated length as fast as any more, and at 32 times the real length the same (bf16, 32
// heads, 30 documents x 160 tokens: re-positioning 13.8 us, 65.9 with a block per piece; assembly 27.8 and 30.6, 87.5 with one).
constexpr int64_t kMostBlocks = 8192;
// Many segments that are re-positioned in several rounds lose up to 6 % by the second (300 x 150 tokens, 32 heads: 142.6 us with a
// block per piece, 151.1 with 8192 blocks, 143.4 with 32768), so there as many blocks as the whole store has pieces, up to this.
constexpr int64_t kMostMoveBlocks = 32768;

template <int DT, int PAIRING>
cf_status launch_dt(const cf_layer_desc* d, const RopeFreq& f, const void* k_in, void* k_out,
                    const cf_segment* segs, int32_t n_seg, int64_t n_store_tokens, int32_t max_seg_len,
                    int32_t* dev_flag, hipStream_t s) {
    const int per_tok = d->n_kv_heads * (d->head_dim / 16);
    const int64_t in_store = n_store_tokens < kMostMoveBlocks * kThreads ? n_store_tokens * per_tok / kThreads + n_seg : kMostMoveBlocks;
    const int64_t most = in_store < kMostBlocks ? kMostBlocks : (in_store > kMostMoveBlocks ? kMostMoveBlocks : in_store);
    const dim3 grid(n_seg, pieces(n_seg, max_seg_len, per_tok, 1, most));
    hipLaunchKernelGGL((reposition_kernel<DT, PAIRING>), grid, dim3(kThreads), 0, s, k_in, k_out, segs, n_store_tokens,
                       d->n_kv_heads, d->head_dim, store_token_stride(d), store_head_stride(d), f, dev_flag, d->max_positions);
    CF_HIP(hipGetLastError());
    return CF_OK;
}

// Final Re-Positioning (Alg. 2, Phase 2): gather + rotate.  grid = (batch * seg_stride, pieces of a segment); block
// (b, s) owns a piece of segment s of query b.  Its output offset is the sum of the visible lengths of the query's
// entries before its own; where it reads depends on its own entry alone, so its first loads are under way while
// the entries are added up and the cos/sin pairs worked out.  Per (token, kv head, 8-pair item) two 16-byte K
// chunks are rotated and two V chunks copied, from the store's (or the own block's) layout to the decode cache's.
template <int DT, int PAIRING, int U>
__global__ __launch_bounds__(kThreads) void assemble_kernel(AssembleArgs a, RopeFreq freq) {
    __shared__ float2 cs[kMaxHalf];
    __shared__ int s_before, s_total, s_bad, s_off_range;
    const int b = (int)div_exact(blockIdx.x, (unsigned)a.seg_stride), s = blockIdx.x - b * a.seg_stride;
    const int tid = threadIdx.x;
    const cf_segment* table = a.segs + (int64_t)b * a.seg_stride;
    // one batch of loads: every index is inside its array whatever the counts turn out to be
    int n = a.n_seg[b];
    const int q0 = a.q_off[b], q1 = a.q_off[b + 1];
    const int64_t q_total = a.q_off[a.batch];
    const int64_t run0 = a.final_off[b];
    const cf_segment seg = table[s];
    const cf_segment mine = table[min(tid, a.seg_stride - 1)];
    if (n < 0 || n > a.seg_stride) {
        if (tid == 0 && s == 0 && blockIdx.y == 0) raise_flag(a.dev_flag, CF_FLAG_BAD_SEGMENT);
        n = n < 0 ? 0 : a.seg_stride;
    }
    if (s >= n && s != 0) return;
    const int tq = min(q1 - q0, a.max_tq);
    // visible tokens of an entry: 0 for a rejected one (bad: malformed; *bad == 2: positions outside the
    // range), min(len, tq) for the own block
    auto visible = [&](const cf_segment& g, int* bad) {
        const bool self = g.kind == CF_SEG_SELF;
        const int64_t limit = self ? q_total : a.n_store_tokens;
        *bad = g.kind < 0 || g.kind > CF_SEG_SELF || g.len < 0 || g.tok_offset < 0 || g.tok_offset + g.len > limit ||
               (self && (a.k_self == nullptr || a.v_self == nullptr));
        if (*bad) return 0;
        const int vis = self ? min(g.len, tq) : g.len;
        if (!positions_ok(g.stored_start, vis, a.max_positions) || !positions_ok(g.new_start, vis, a.max_positions)) *bad = 2;
        return *bad ? 0 : vis;
    };
    int bad;
    const int vis = s < n ? visible(seg, &bad) : 0;
    const bool self = seg.kind == CF_SEG_SELF;
    const int half = a.head_dim >> 1;
    const int items_per_head = half / 8;                 // head_dim % 16 == 0 checked on the host
    const void* k_in = self ? a.k_self : a.k_store;
    const void* v_in = self ? a.v_self : a.v_store;
    const int64_t in_ts = self ? (int64_t)a.n_kv_heads * a.head_dim : a.store_ts;
    const int64_t in_hs = self ? a.head_dim : a.store_hs;
    const bool by_head = a.final_hs > a.final_ts;
    Walk<U> walk(vis, a.n_kv_heads * items_per_head);
    const int delta = seg.new_start - seg.stored_start;
    // adds up the query's entries (before its own, in all) and, in the query's first block, reports them
    auto add_up = [&]() {
        if (tid == 0) { s_before = 0; s_total = 0; s_bad = 0; s_off_range = 0; }
        __syncthreads();
        for (int t = tid; t < n; t += kThreads) {
            int wrong;
            const int len = visible(t == tid ? mine : table[t], &wrong);
            if (wrong == 1) atomicOr(&s_bad, 1);
            if (wrong == 2) atomicOr(&s_off_range, 1);
            atomicAdd(&s_total, len);
            if (t < s) atomicAdd(&s_before, len);
        }
        if (delta != 0)
            for (int m = tid; m < half; m += kThreads) cs[m] = rope_cos_sin(delta, freq.rev[m]);
        __syncthreads();
        const bool fits = run0 >= 0 && run0 + s_total <= a.final_capacity;
        if (s == 0 && blockIdx.y == 0 && tid == 0) {
            if (s_bad) raise_flag(a.dev_flag, CF_FLAG_BAD_SEGMENT);
            if (s_off_range) raise_flag(a.dev_flag, CF_FLAG_POS_RANGE);
            if (!fits) raise_flag(a.dev_flag, CF_FLAG_BAD_INDEX);
            a.final_len[b] = fits ? s_total : 0;
        }
        return fits;
    };
    if (!walk.more()) {                                  // nothing to move
        if (s == 0 && blockIdx.y == 0) add_up();
        return;
    }
    bool first = true;
    int64_t out0 = 0;
    for (; walk.more(); walk.next()) {
        const int n_items = walk.n_items();
        Chunk8<DT> x[U], y[U], va[U], vb[U];
        int tok[U], head[U], j[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // an item past the end reads the last one again and stores nothing
            const Item i = locate(min(walk.at + u * kThreads + tid, n_items - 1), items_per_head, a.n_kv_heads, walk.ntok(), by_head);
            tok[u] = walk.tok0 + i.tok;
            head[u] = i.head;
            j[u] = i.j;
            const int64_t src = (seg.tok_offset + tok[u]) * in_ts + (int64_t)i.head * in_hs;
            const int o0 = first_of<PAIRING>(i.j), o1 = second_of<PAIRING>(i.j, half);
            x[u].load(k_in, src + o0);
            y[u].load(k_in, src + o1);
            va[u].load(v_in, src + o0);
            vb[u].load(v_in, src + o1);
        }
        if (first) {
            if (!add_up()) return;                       // the whole block
            out0 = run0 + s_before;
            first = false;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (walk.at + u * kThreads + tid >= n_items) continue;
            const int64_t dst = (out0 + tok[u]) * a.final_ts + (int64_t)head[u] * a.final_hs;
            const int o0 = first_of<PAIRING>(j[u]), o1 = second_of<PAIRING>(j[u], half);
            if (delta != 0) rotate<DT, PAIRING>(x[u], y[u], cs, j[u]);
            x[u].template store<kStream<DT>>(a.k_final, dst + o0);
            y[u].template store<kStream<DT>>(a.k_final, dst + o1);
            va[u].template store<kStream<DT>>(a.v_final, dst + o0);
            vb[u].template store<kStream<DT>>(a.v_final, dst + o1);
            if (a.final_pos && j[u] == 0 && head[u] == 0) a.final_pos[out0 + tok[u]] = seg.new_start + tok[u];
        }
    }
}

template <int DT, int PAIRING, int U>
cf_status launch_assemble_piece(const cf_layer_desc* d, const RopeFreq& f, const AssembleArgs& a, int32_t max_seg_len,
                                hipStream_t s) {
    const int64_t entries = (int64_t)a.batch * a.seg_stride;
    // every block adds up its query's whole table, so the longer the table the fewer blocks (bf16, 8 heads, 1000 / 2000 documents x 10-30
    // tokens: 85.5 -> 62.9 and 278 -> 127 us; up to 300 entries no difference)
    const int64_t most = a.seg_stride > kThreads ? kMostBlocks * kThreads / a.seg_stride : kMostBlocks;
    const dim3 grid((unsigned)entries, pieces(entries, max_seg_len, d->n_kv_heads * (d->head_dim / 16), U, most));
    hipLaunchKernelGGL((assemble_kernel<DT, PAIRING, U>), grid, dim3(kThreads), 0, s, a, f);
    CF_HIP(hipGetLastError());
    return CF_OK;
}

template <int DT, int PAIRING>
cf_status launch_assemble_dt(const cf_layer_desc* d, const RopeFreq& f, const AssembleArgs& a, int32_t max_seg_len,
                             hipStream_t s) {
    // Two items per thread share a block's table sums and cos/sin pairs, but leave half as many blocks.  From 1024 blocks of
    // one on they are faster (30 documents x 160 tokens of 32 heads, bf16: 33.7 against 35.8 us; 5 queries x 7
    // documents of 199 and more tokens, 4 heads: 10.6 against 10.9), below it slower (under 7 us: by 0.1-0.5 us).
    const int64_t items = (int64_t)a.batch * a.seg_stride * max_seg_len * d->n_kv_heads * (d->head_dim / 16);
    if (items < (int64_t)256 * 4 * kThreads) return launch_assemble_piece<DT, PAIRING, 1>(d, f, a, max_seg_len, s);
    return launch_assemble_piece<DT, PAIRING, 2>(d, f, a, max_seg_len, s);
}

template <class F> cf_status by_pairing(const cf_layer_desc* d, F&& go) {
    return d->rope_pairing == CF_ROPE_HALF ? go(std::integral_constant<int, CF_ROPE_HALF>{})
                                           : go(std::integral_constant<int, CF_ROPE_INTERLEAVED>{});
}

}  // namespace

cf_status launch_assemble(const cf_layer_desc* d, const RopeFreq& f, const AssembleArgs& a, int32_t max_seg_len,
                          hipStream_t s) {
    switch (d->dtype) {
        case CF_F32: return by_pairing(d, [&](auto P) { return launch_assemble_dt<CF_F32, P.value>(d, f, a, max_seg_len, s); });
        case CF_BF16: return by_pairing(d, [&](auto P) { return launch_assemble_dt<CF_BF16, P.value>(d, f, a, max_seg_len, s); });
        default: return by_pairing(d, [&](auto P) { return launch_assemble_dt<CF_F16, P.value>(d, f, a, max_seg_len, s); });
    }
}

cf_status launch_reposition(const cf_layer_desc* d, const RopeFreq& f, const void* k_in, void* k_out,
                            const cf_segment* segs, int32_t n_seg, int64_t n_store_tokens,
                            int32_t max_seg_len, int32_t* dev_flag, hipStream_t s) {
    switch (d->dtype) {
        case CF_F32: return by_pairing(d, [&](auto P) { return launch_dt<CF_F32, P.value>(d, f, k_in, k_out, segs, n_seg, n_store_tokens, max_seg_len, dev_flag, s); });
        case CF_BF16: return by_pairing(d, [&](auto P) { return launch_dt<CF_BF16, P.value>(d, f, k_in, k_out, segs, n_seg, n_store_tokens, max_seg_len, dev_flag, s); });
        default: return by_pairing(d, [&](auto P) { return launch_dt<CF_F16, P.value>(d, f, k_in, k_out, segs, n_seg, n_store_tokens, max_seg_len, dev_flag, s); });
    }
}

}  // namespace cf
