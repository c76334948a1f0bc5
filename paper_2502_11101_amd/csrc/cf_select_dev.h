// Device-side building blocks of the integer side of Layer-Adaptive Cache Pruning: ranking
// (Alg. 2, argsort + prun), position allocation (Eq. 6, Sec. 2.5) and the segment-table rebuild
// (the logical concat of Alg. 2), each executed by one workgroup for one query.  They are used
// by the stand-alone kernels behind cf_prune_topk / cf_assign_positions / cf_gather_segments and
// by the fused layer epilogue.  Candidate sets are small (tens to a few hundred documents), so
// ranking is by counting with exact comparisons: results do not depend on thread order.
#pragma once

#include "cf_common.h"

namespace cf {

// true when candidate (score sa, len la, slot ia, list position pa) ranks before (sb, lb, ib, pb):
// higher score/len first, compared as sa*lb vs sb*la in fp64 (exact: 24-bit significand times an
// integer below 2^24 fits 53 bits), then lower slot, then earlier list position.
__device__ __forceinline__ bool ranks_before(float sa, int la, int ia, int pa, float sb, int lb, int ib, int pb) {
    const double x = (double)sa * (double)lb;
    const double y = (double)sb * (double)la;
    if (x != y) return x > y;
    if (ia != ib) return ia < ib;
    return pa < pb;
}

// The three functions below are called by the first `nthr` threads of a workgroup, all of them, and by
// no others; when the workgroup's other wavefronts have exited, nthr is one wavefront and the barriers
// inside cost nothing.
//
// smem: 3*stride 32-bit words.  Returns the number kept (0 after a flagged error).
// score/len/cand/keep_idx point at this query's rows.
__device__ inline int prune_topk_block(const float* score, const int32_t* len, const int32_t* cand, int n, int keep,
                                       int stride, int32_t* keep_idx, int32_t* dev_flag, unsigned char* smem,
                                       int* s_bad, int nthr) {
    float* s_score = reinterpret_cast<float*>(smem);
    int32_t* s_len = reinterpret_cast<int32_t*>(s_score + stride);
    int32_t* s_idx = s_len + stride;
    const int tid = threadIdx.x;
    if (tid == 0) *s_bad = 0;
    __syncthreads();
    if (n < 0 || n > stride) {
        if (tid == 0) raise_flag(dev_flag, CF_FLAG_BAD_INDEX);
        return 0;
    }
    for (int i = tid; i < n; i += nthr) {
        const int c = cand[i];
        int flag = 0;
        float sc = 0.f;
        int ln = 1;
        if (c < 0 || c >= stride) {
            flag = CF_FLAG_BAD_INDEX;
        } else {
            sc = score[c];
            ln = len ? len[c] : 1;
            if (!isfinite(sc)) flag = CF_FLAG_NONFINITE_SCORE;
            if (ln <= 0 || ln >= (1 << 24)) flag |= CF_FLAG_BAD_SEGMENT;
        }
        if (flag) atomicOr(s_bad, flag);
        s_score[i] = sc;
        s_len[i] = ln;
        s_idx[i] = c;
    }
    __syncthreads();
    if (*s_bad) {
        if (tid == 0) raise_flag(dev_flag, *s_bad);
        return 0;
    }
    const int k = min(keep, n);
    for (int i = tid; i < n; i += nthr) {
        const float si = s_score[i];
        const int li = s_len[i], ci = s_idx[i];
        int rank = 0;
        for (int j = 0; j < n; ++j)
            rank += (j != i) && ranks_before(s_score[j], s_len[j], s_idx[j], j, si, li, ci, i);
        if (rank < k) keep_idx[rank] = ci;
    }
    return k;
}

// smem: 3*stride 32-bit words; s_int: 3 ints of LDS.  Pointers are this query's rows; q_start /
// n_reuse point at this query's entries.  Returns false (outputs untouched) after a flagged error.
__device__ inline bool assign_positions_block(const int32_t* len, const int32_t* ranked, int n, int stride, int pos_begin,
                                              int pos_end, int strategy, int force_n_reuse, int32_t* new_start,
                                              int32_t* q_start, int32_t* n_reuse, int32_t* order, int32_t* dev_flag,
                                              unsigned char* smem, int* s_int, int nthr) {
    int32_t* s_ord = reinterpret_cast<int32_t*>(smem);   // placement order (slots)
    int32_t* s_len = s_ord + stride;                      // length per placement rank
    int32_t* s_cum = s_len + stride;                      // distance from the query to the start
    int &bad = s_int[0], &lmax = s_int[1], &span_max = s_int[2];
    const int tid = threadIdx.x;
    __syncthreads();
    if (tid == 0) { bad = 0; lmax = 0; span_max = 0; }
    __syncthreads();
    if (n < 0 || n > stride) {
        if (tid == 0) raise_flag(dev_flag, CF_FLAG_BAD_INDEX);
        return false;
    }
    // placement order: as ranked ("sort") or by ascending slot ("align", and the listing order of "keep")
    for (int i = tid; i < n; i += nthr) {
        const int c = ranked[i];
        if (c < 0 || c >= stride) atomicOr(&bad, CF_FLAG_BAD_INDEX);
        s_cum[i] = c;
    }
    __syncthreads();
    if (bad) {
        if (tid == 0) raise_flag(dev_flag, bad);
        return false;
    }
    for (int i = tid; i < n; i += nthr) {
        const int c = s_cum[i];
        int r = i;
        if (strategy != CF_ALLOC_SORT) {
            r = 0;
            for (int j = 0; j < n; ++j) {
                const int cj = s_cum[j];
                r += (cj < c) || (cj == c && j < i);
            }
        }
        s_ord[r] = c;
    }
    __syncthreads();
    for (int i = tid; i < n; i += nthr) {
        const int l = len[s_ord[i]];
        s_len[i] = l;
        if (l <= 0) atomicOr(&bad, CF_FLAG_BAD_SEGMENT);
        atomicMax(&lmax, l);
    }
    __syncthreads();
    if (bad) {
        if (tid == 0) raise_flag(dev_flag, bad);
        return false;
    }
    if (strategy == CF_ALLOC_KEEP || n == 0) {
        for (int i = tid; i < n; i += nthr) order[i] = s_ord[i];
        if (n == 0 && strategy != CF_ALLOC_KEEP && tid == 0) { *q_start = pos_begin; *n_reuse = 0; }
        return true;
    }
    const int avail = pos_end - pos_begin;
    const int cap = avail / lmax;
    if (cap <= 0) {
        if (tid == 0) raise_flag(dev_flag, CF_FLAG_DOC_TOO_LONG);
        return false;
    }
    int groups = force_n_reuse > 0 ? force_n_reuse : (n + cap - 1) / cap;
    groups = min(groups, n);
    const int per_group = (n + groups - 1) / groups;
    for (int i = tid; i < n; i += nthr) {
        const int first = (i / per_group) * per_group;
        int cum = 0;
        for (int j = first; j <= i; ++j) cum += s_len[j];
        s_cum[i] = cum;
        const bool last = (i == n - 1) || ((i + 1) % per_group == 0);
        if (last) atomicMax(&span_max, cum);
    }
    __syncthreads();
    if (span_max > avail) {
        if (tid == 0) raise_flag(dev_flag, CF_FLAG_POS_OVERFLOW);
        return false;
    }
    const int qs = pos_begin + span_max;
    for (int i = tid; i < n; i += nthr) {
        new_start[s_ord[i]] = qs - s_cum[i];
        order[i] = s_ord[i];
    }
    if (tid == 0) { *q_start = qs; *n_reuse = groups; }
    return true;
}

// doc_tok_offset/len/order/new_start point at this query's rows, out at this query's segment-table
// row.  q_lo/q_hi: this query's rows in q.
__device__ inline void gather_segments_block(const int64_t* doc_tok_offset, const int32_t* len, const int32_t* order, int n,
                                             const int32_t* new_start, int q_start, int q_lo, int q_hi, int stride,
                                             int prefix_len, int doc_stored_start, int q_stored_start, cf_segment* out,
                                             int32_t* n_seg, int seg_stride, int32_t* dev_flag, int nthr) {
    const int tid = threadIdx.x;
    const int has_prefix = prefix_len > 0 ? 1 : 0;
    if (n < 0 || n > stride || n + has_prefix + 1 > seg_stride) {
        if (tid == 0) { raise_flag(dev_flag, CF_FLAG_BAD_INDEX); *n_seg = 0; }
        return;
    }
    if (tid == 0) {
        if (has_prefix) {
            cf_segment p;
            p.tok_offset = 0; p.len = prefix_len; p.stored_start = 0; p.new_start = 0;
            p.kind = CF_SEG_PREFIX; p.doc = -1; p.reserved = 0;
            out[0] = p;
        }
        cf_segment q;
        q.tok_offset = q_lo; q.len = q_hi - q_lo; q.stored_start = q_stored_start;
        q.new_start = q_start; q.kind = CF_SEG_SELF; q.doc = -1; q.reserved = 0;
        out[has_prefix + n] = q;
        *n_seg = has_prefix + n + 1;
    }
    for (int i = tid; i < n; i += nthr) {
        const int c = order[i];
        cf_segment sgm;
        if (c < 0 || c >= stride) {
            raise_flag(dev_flag, CF_FLAG_BAD_INDEX);
            sgm.tok_offset = 0; sgm.len = 0; sgm.stored_start = 0; sgm.new_start = 0;
            sgm.kind = CF_SEG_DOC; sgm.doc = -1; sgm.reserved = 0;
        } else {
            sgm.tok_offset = doc_tok_offset[c]; sgm.len = len[c];
            sgm.stored_start = doc_stored_start; sgm.new_start = new_start[c];
            sgm.kind = CF_SEG_DOC; sgm.doc = c; sgm.reserved = 0;
        }
        out[has_prefix + i] = sgm;
    }
}

// ---------------------------------------------------------------------------------------------
// The same three stages for at most 64 candidates, every list in registers (lane i = list position i).  A lane issues one instruction at a time
// and each of a chain waits for the one before, so what can be is spread over the workgroup: the ranking, which is most of it, over all
// wavefronts but one (rank_share), the rest — permutes, sums and maxima across the lanes — by one (select_wave64), without barriers or
// atomics.  Results are those of the block functions; on any condition they would flag (bad
// index, non-finite score, bad length, document too long, overflow, table too small) nothing is
// written and false is returned, so that the caller runs the block functions, which raise the flag.
// On one wavefront alone, with its lists handed over through LDS, this took 3000 cycles for ten candidates and 6200 for fifty; now 2600 and 3700.
struct SelectWaveArgs {
    const float* score; const int32_t* len; const int32_t* cand; const int64_t* tok; const int32_t* start;      // the query's rows, in LDS
    int32_t* keep_idx; int32_t* new_start; int32_t* order;                                                      // its rows in memory
    int n, keep, stride, normalise_by_len, strategy, force_n_reuse, pos_begin, pos_end;
    int prefix_len, doc_stored_start, q_stored_start, q_lo, q_hi, seg_stride;
    int q_start, n_reuse;                           // as they stand ("keep" leaves them)
};

__device__ __forceinline__ int lane_int(int v, int from) { return __builtin_amdgcn_readlane(v, from); }

// list position `lane`'s candidate; `bad` (any of the list's): the block functions' business.  tok and start: of the candidate.
struct Candidate { int c, len, start; int64_t tok; bool have, bad; };
__device__ inline Candidate load_candidate(const SelectWaveArgs& s) {
    const int lane = threadIdx.x & 63;
    Candidate d;
    d.have = lane < min(s.n, s.stride);
    d.c = d.have ? s.cand[lane] : 0;
    const bool c_ok = d.c >= 0 && d.c < s.stride;
    const int at = c_ok ? d.c : 0;
    const float sc = s.score[at];
    d.len = s.len[at];
    d.start = s.start[at];
    d.tok = s.tok[at];
    const int ln = s.normalise_by_len ? d.len : 1;
    d.bad = __any(d.have && (!c_ok || !isfinite(sc) || ln <= 0 || ln >= (1 << 24))) || s.n < 0 || s.n > 64 || s.n > s.stride;
    return d;
}

// Ranking (Alg. 2: argsort of the accumulated scores).  A wavefront compares every candidate (lane i = list position i) with its share of
// them, as ranks_before does, and adds to rank[i] (LDS, cleared) how many of those rank before it.  What does not wait for the scores, before
// they are there.  (Of lists that load_candidate calls bad the ranks mean nothing.)
constexpr int kRankShare = 5;                       // at most 64 candidates, at least 13 wavefronts
struct RankShare { int at, j[kRankShare]; double len, len_j[kRankShare]; bool have, tie[kRankShare]; };
__device__ inline RankShare rank_prepare(const SelectWaveArgs& s, int wave, int n_waves) {
    const int lane = threadIdx.x & 63;
    RankShare r;
    r.have = lane < min(s.n, s.stride);
    const int c = r.have ? s.cand[lane] : 0;
    r.at = c >= 0 && c < s.stride ? c : 0;
    const int ln = s.normalise_by_len ? s.len[r.at] : 1;
    r.len = (double)ln;
#pragma unroll
    for (int i = 0; i < kRankShare; ++i) {
        const int j = wave + i * n_waves;
        r.j[i] = j < min(s.n, 64) ? j : -1;
        if (r.j[i] < 0) continue;
        const int cj = lane_int(c, j);
        r.len_j[i] = (double)lane_int(ln, j);
        r.tie[i] = cj != c ? cj < c : j < lane;         // lower slot, then earlier list position
    }
    return r;
}
__device__ inline void rank_share(const SelectWaveArgs& s, const RankShare& r, int32_t* rank) {
    if (r.j[0] < 0) return;
    const float score = s.score[r.at];
    const double sc = (double)score;
    int before = 0;
#pragma unroll
    for (int i = 0; i < kRankShare; ++i) {
        if (r.j[i] < 0) continue;
        const double x = (double)__int_as_float(lane_int(__float_as_int(score), r.j[i])) * r.len, y = sc * r.len_j[i];
        before += x > y || (x == y && r.tie[i]) ? 1 : 0;
    }
    if (r.have) atomicAdd(rank + (threadIdx.x & 63), before);
}

// In-register reductions over the 64 lanes of a wavefront with DPP (row shifts, then the two row broadcasts,
// lane 63 ends up with the result): an inclusive prefix sum, and a maximum handed to every lane.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
    return v;
}

__device__ __forceinline__ int wave_max_i32(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(v, 63);
}

// The cut, the allocation and the next table, by one wavefront with all its lanes; `rank`: of the lane's candidate.
__device__ inline bool select_wave64(const SelectWaveArgs& s, const Candidate& cd, int rank, int32_t* n_keep_out, int32_t* q_start_out,
                                     int32_t* n_reuse_out, cf_segment* out, int32_t* n_seg_out) {
    const int lane = threadIdx.x & 63;
    const int n = s.n;
    if (cd.bad) return false;
    const int k = min(s.keep, n);
    const int has_prefix = s.prefix_len > 0 ? 1 : 0;
    if (k + has_prefix + 1 > s.seg_stride) return false;
    const bool in = lane < k;
    // ranked list: lane r gets the candidate of rank r (the ranks of the n lanes are 0 .. n - 1; the others keep their places)
    auto move = [](int to, int v) { return __builtin_amdgcn_ds_permute(to << 2, v); };
    const int64_t tok = cd.tok;
    const int to = cd.have ? rank : lane;
    const int rc = move(to, cd.c);
    int oc = rc, pl = move(to, cd.len), my_start = move(to, cd.start);
    int tok_lo = move(to, (int)(uint32_t)tok), tok_hi = move(to, (int)(uint32_t)((uint64_t)tok >> 32));
    // ---- placement order (Sec. 2.5): as ranked ("sort") or by ascending slot ("align"; listing order of "keep")
    if (s.strategy != CF_ALLOC_SORT) {
        int place = 0;
        for (int j = 0; j < k; ++j) {
            const int cj = lane_int(rc, j);
            place += (cj < rc) || (cj == rc && j < lane);
        }
        place = in ? place : lane;
        oc = move(place, rc);
        pl = move(place, pl);
        my_start = move(place, my_start);
        tok_lo = move(place, tok_lo);
        tok_hi = move(place, tok_hi);
    }
    if (__any(in && pl <= 0)) return false;
    pl = in ? pl : 0;
    int qs = s.q_start, groups = s.n_reuse;
    bool write_pos = false;
    if (s.strategy != CF_ALLOC_KEEP && k > 0) {
        // ---- allocation (Eq. 6): capacity by the longest survivor, balanced contiguous groups, every group
        // ends at the query
        const int lmax = wave_max_i32(pl);
        const int avail = s.pos_end - s.pos_begin;
        if (lmax > avail) return false;                   // (capacity avail / lmax; lmax >= 1: every kept length is positive)
        groups = s.force_n_reuse;
        if (groups <= 0) {
            groups = 1;
            if ((int64_t)lmax * k > avail) {              // the capacity is less than all
                const int cap = (int)div_exact((unsigned)avail, (unsigned)lmax);
                groups = (int)div_exact((unsigned)(k + cap - 1), (unsigned)cap);
            }
        }
        groups = min(groups, k);
        int cum = wave_inclusive_scan(pl);                // inclusive prefix over placement ranks
        int span_max = lane_int(cum, 63);                 // (one group: all of it)
        if (groups > 1) {
            const int per_group = (int)div_exact((unsigned)(k + groups - 1), (unsigned)groups);
            const int first = (int)div_exact((unsigned)lane, (unsigned)per_group) * per_group;
            const int before = __shfl(cum, max(first - 1, 0));
            cum -= first > 0 ? before : 0;
            const bool last = in && ((lane == k - 1) || (lane + 1 == first + per_group));
            span_max = wave_max_i32(last ? cum : 0);
        }
        if (span_max > avail) return false;
        qs = s.pos_begin + span_max;
        my_start = qs - cum;
        write_pos = true;
    } else if (s.strategy != CF_ALLOC_KEEP) {             // nothing survives
        qs = s.pos_begin;
        groups = 0;
    }
    // ---- everything checked: write the lists and the next segment table (Alg. 2, the logical concat)
    if (in) {
        cf_segment sg;
        sg.tok_offset = (int64_t)((uint64_t)(uint32_t)tok_hi << 32 | (uint32_t)tok_lo);
        sg.len = pl; sg.stored_start = s.doc_stored_start; sg.new_start = my_start;
        sg.kind = CF_SEG_DOC; sg.doc = oc; sg.reserved = 0;
        out[has_prefix + lane] = sg;
        s.keep_idx[lane] = rc;
        s.order[lane] = oc;
        if (write_pos) s.new_start[oc] = my_start;
    }
    if (lane == 0) {
        *n_keep_out = k;
        if (s.strategy != CF_ALLOC_KEEP) { *q_start_out = qs; *n_reuse_out = groups; }
        if (has_prefix) {
            cf_segment p;
            p.tok_offset = 0; p.len = s.prefix_len; p.stored_start = 0; p.new_start = 0;
            p.kind = CF_SEG_PREFIX; p.doc = -1; p.reserved = 0;
            out[0] = p;
        }
        cf_segment q;
        q.tok_offset = s.q_lo; q.len = s.q_hi - s.q_lo; q.stored_start = s.q_stored_start;
        q.new_start = qs; q.kind = CF_SEG_SELF; q.doc = -1; q.reserved = 0;
        out[has_prefix + k] = q;
        *n_seg_out = has_prefix + k + 1;
    }
    return true;
}

}  // namespace cf
