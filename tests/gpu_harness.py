"""GPU-side glue for the parity tests: upload a synthetic workload, run the library through
its C ABI (via the binding), fetch results, and compute the error metrics."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from oracle import cachefocus_oracle as orc
from paper_2502_11101_amd import binding as cf
from paper_2502_11101_amd import pipeline as pl
from paper_2502_11101_amd import workloads as wl
from tests import helpers as H

OUT_TOL = {"f32": 1e-4, "bf16": 2e-2, "f16": 2e-2}
MASS_TOL = {"f32": 1e-5, "bf16": 1e-4, "f16": 1e-4}
# Masses against the rounded-key reference (helpers.rounded_key_reference) on shapes with few rows and short
# documents: 1e-4 for the kernels' own arithmetic plus as much again for key elements that the kernels' fp32
# rotation (hardware sine/cosine) rounds to the other 16-bit neighbour than the reference's fp64 rotation does — a
# few elements in a thousand, each moving one score by a 16-bit step.  (Seen over all such tests: at most 1.2e-4.)
NEAR_MASS_TOL = {"f32": 1e-5, "bf16": 2e-4, "f16": 2e-4}


def rounds_moved_keys(g, pairing, seg_stride) -> bool:
    """Whether a call of this shape takes the 16-bit MFMA kernels, which round a moved key once to the storage
    type (the others turn the query, or the keys on the fly, in fp32 and round nothing)."""
    return g.dtype != "f32" and g.head_dim == 128 and pairing == cf.CF_ROPE_HALF and seg_stride <= 256


# store layouts exercised by the tests: token-major, head-major, head-major with unused rows per head
LAYOUTS = {"token": ("token", 0), "head": ("head", 0), "head_padded": ("head", 5)}


def desc_of(cfg: wl.Config, pairing=cf.CF_ROPE_HALF, layout="token", n_store_tokens=0):
    g = cfg.geometry
    kind, pad = LAYOUTS[layout]
    ts, hs = (0, 0) if layout == "token" else pl.store_strides(n_store_tokens, g.n_kv_heads, g.head_dim, kind, pad)
    return cf.make_desc(g.n_q_heads, g.n_kv_heads, g.head_dim, g.dtype, g.rope_base, g.max_positions, pairing,
                        store_token_stride=ts, store_head_stride=hs)


def upload_layer(cfg: wl.Config, tensors: dict, layout="token"):
    g = cfg.geometry
    kind, pad = LAYOUTS[layout]
    return {k: (pl.store_to_device(v, g.dtype, kind, pad) if k in ("k_store", "v_store") else pl.to_device(v, g.dtype))
            for k, v in tensors.items()}


def make_batch(cfg: wl.Config, st: wl.Structure, pairing=cf.CF_ROPE_HALF, layout="token") -> pl.PrefillBatch:
    off = st.doc_off[:-1][st.query_docs]                 # [batch, k]
    lens = st.doc_lens[st.query_docs]
    return pl.PrefillBatch(desc_of(cfg, pairing, layout, st.n_store_tokens), off, lens, cfg.tq, cfg.prefix_len,
                           cfg.doc_stored_start, st.n_store_tokens)


def row_error(gpu: np.ndarray, ref: np.ndarray) -> float:
    """max over (row, head) of ||gpu - ref||_inf / ||ref[row, head]||_inf."""
    diff = np.abs(gpu.astype(np.float64) - ref).max(axis=-1)
    norm = np.abs(ref).max(axis=-1)
    return float((diff / norm).max())


def rel_error(gpu: np.ndarray, ref: np.ndarray) -> float:
    ref = np.asarray(ref, dtype=np.float64)
    return float((np.abs(gpu.astype(np.float64) - ref) / np.maximum(np.abs(ref), 1e-300)).max())


def device_segments(pb: pl.PrefillBatch, b: int):
    """Query b's current segment table as oracle Segment tuples."""
    n = int(pb.n_seg[b].item())
    arr = cf.segments_from_device(pb.segs[b], n)
    return [orc.Segment(int(r["tok_offset"]), int(r["len"]), int(r["stored_start"]), int(r["new_start"]),
                        int(r["kind"]), int(r["doc"])) for r in arr]


def oracle_on_device_segments(cfg: wl.Config, tensors: dict, pb: pl.PrefillBatch, b: int, pairing="half"):
    """Run the oracle for query b on exactly the segment table the device holds."""
    g = cfg.geometry
    segs = device_segments(pb, b)
    q_start = int(pb.q_start[b].item())
    q = np.asarray(tensors["q"][b * cfg.tq:(b + 1) * cfg.tq], dtype=np.float64)
    out, mass = orc.prefill_attention(q, pb.q_stored_start, q_start, tensors["k_store"], tensors["v_store"],
                                      tensors["k_self"], tensors["v_self"], segs, g.n_kv_heads, g.rope_base,
                                      pairing)
    return segs, out, mass


def check_tables(hq, hkv, tq, tables, n_store, dtype, q_pos, seed, layout="head", lengths=None, check=None, shape=None, given=None, own_first=False):
    """cf_prefill_attention on hand-written tables against the oracle, with masses and without (the same outputs, bit for bit).
    `tables`: per query the (offset, length, stored, new) of its store segments; the own block of the query's rows follows (own_first:
    comes before them) at q_pos.
    `lengths`: rows per query where they are not all tq; `check`: the queries compared (default: all); `shape(tensors, rng)` may
    replace what was drawn; `given`: the workspace's bytes where they are not those reported for the call."""
    rng = np.random.default_rng(seed)
    batch = len(tables)
    lengths = [tq] * batch if lengths is None else list(lengths)
    q_off = np.concatenate([[0], np.cumsum(lengths)]).astype(int)
    normal = lambda n, h: wl.round_to_dtype(rng.standard_normal((n, h, 128), dtype=np.float32), dtype)
    rows_all = int(q_off[-1])
    t = dict(q=normal(rows_all, hq), k_self=normal(rows_all, hkv), v_self=normal(rows_all, hkv), k_store=normal(n_store, hkv),
             v_store=normal(n_store, hkv))
    if shape is not None:
        shape(t, rng)
    dev = {k: (pl.store_to_device(v, dtype, layout, 0) if k in ("k_store", "v_store") else pl.to_device(v, dtype)) for k, v in t.items()}
    ts, hs = (0, 0) if layout == "token" else pl.store_strides(n_store, hkv, 128, layout, 0)
    desc = cf.make_desc(hq, hkv, 128, dtype, 1.0e4, 8192, cf.CF_ROPE_HALF, store_token_stride=ts, store_head_stride=hs)
    stride = max(len(x) for x in tables) + 1
    rows, segs = [], []
    for b, x in enumerate(tables):
        own = [orc.Segment(o, n, s, p, orc.KIND_DOC, i) for i, (o, n, s, p) in enumerate(x)] + \
            [orc.Segment(int(q_off[b]), lengths[b], 0, q_pos, orc.KIND_SELF, -1)]
        own = own[-1:] + own[:-1] if own_first else own
        segs.append(own)
        rows += [(g.tok_offset, g.len, g.stored_start, g.new_start, g.kind, g.doc) for g in own]
        rows += [(0, 0, 0, 0, cf.CF_SEG_DOC, -1)] * (stride - len(own))
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    table = cf.segments_to_device(cf.segments_array(rows))
    max_kv = max(sum(n for _, n, _, _ in x) for x in tables) + tq
    need = cf.cf_prefill_workspace_bytes(desc, batch, tq, stride, max_kv) if given is None else given
    ws = torch.full((need + 4096,), 0xFF, dtype=torch.uint8, device="cuda")      # what follows the workspace is not touched
    flag, out = i32([0]), torch.empty_like(dev["q"])
    args = (desc, dev["q"], i32(q_off.tolist()), 0, i32([q_pos] * batch), dev["k_store"], dev["v_store"], n_store, dev["k_self"],
            dev["v_self"], table, i32([len(x) for x in segs]), stride, batch, tq, max_kv)
    cf.cf_prefill_attention(*args, out, None, None, 1, ws, need, flag)
    ws.fill_(0xFF)
    again, mass = torch.empty_like(out), torch.zeros((batch, stride), dtype=torch.float32, device="cuda")
    cf.cf_prefill_attention(*args, again, mass, None, 1, ws, need, flag)
    torch.cuda.synchronize()
    assert int(flag.item()) == 0 and torch.equal(again, out) and bool((ws[need:] == 0xFF).all())
    got, mass = out.float().cpu().numpy(), mass.cpu().numpy()
    assert np.isfinite(got).all() and np.isfinite(mass).all()
    for b in range(batch) if check is None else check:
        if lengths[b] == 0:
            continue
        part = slice(q_off[b], q_off[b + 1])
        ks, vs, compact = H.compact_query(segs[b], t["k_store"], t["v_store"]) if len(segs[b]) > 1 else (None, None, segs[b])
        ref, near = H.rounded_key_reference(dtype, t["q"][part], 0, q_pos, ks, vs, t["k_self"], t["v_self"], compact, hkv, 1.0e4)
        assert row_error(got[part], ref) <= OUT_TOL[dtype], b
        assert rel_error(mass[b, :len(segs[b])], near) <= NEAR_MASS_TOL[dtype], b
        assert mass[b].sum() == pytest.approx(hq * lengths[b], rel=1e-5), b
