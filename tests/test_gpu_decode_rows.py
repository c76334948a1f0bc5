"""GPU parity of the attention kernel for one 16-row block (decode steps): every wavefront streams tiles of its own.
Tile counts from fewer than the wavefronts to several each, ragged ends, several splits and one, moved and unmoved keys, rows from one
to sixteen with the causal own block, and the longer tables that the other kernel keeps."""

import numpy as np
import pytest
import torch

from paper_2502_11101_amd import binding as cf
from paper_2502_11101_amd import pipeline as pl
from paper_2502_11101_amd import workloads as wl
from tests import gpu_harness as G
from tests import helpers as H
from oracle import cachefocus_oracle as orc

pytestmark = pytest.mark.gpu


def _check(hq, hkv, tq, tables, n_store, dtype, q_pos, seed, layout="head"):
    """`tables`: per query the (offset, length, stored, new) of its store segments; the own block of tq rows follows at q_pos."""
    rng = np.random.default_rng(seed)
    batch = len(tables)
    normal = lambda n, h: wl.round_to_dtype(rng.standard_normal((n, h, 128), dtype=np.float32), dtype)
    t = dict(q=normal(batch * tq, hq), k_self=normal(batch * tq, hkv), v_self=normal(batch * tq, hkv), k_store=normal(n_store, hkv),
             v_store=normal(n_store, hkv))
    dev = {k: (pl.store_to_device(v, dtype, layout, 0) if k in ("k_store", "v_store") else pl.to_device(v, dtype)) for k, v in t.items()}
    ts, hs = (0, 0) if layout == "token" else pl.store_strides(n_store, hkv, 128, layout, 0)
    desc = cf.make_desc(hq, hkv, 128, dtype, 1.0e4, 8192, cf.CF_ROPE_HALF, store_token_stride=ts, store_head_stride=hs)
    stride = max(len(x) for x in tables) + 1
    rows, segs = [], []
    for b, x in enumerate(tables):
        own = [orc.Segment(o, n, s, p, orc.KIND_DOC, i) for i, (o, n, s, p) in enumerate(x)] + \
            [orc.Segment(b * tq, tq, 0, q_pos, orc.KIND_SELF, -1)]
        segs.append(own)
        rows += [(g.tok_offset, g.len, g.stored_start, g.new_start, g.kind, g.doc) for g in own]
        rows += [(0, 0, 0, 0, cf.CF_SEG_DOC, -1)] * (stride - len(own))
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    table = cf.segments_to_device(cf.segments_array(rows))
    max_kv = max(sum(n for _, n, _, _ in x) for x in tables) + tq
    need = cf.cf_prefill_workspace_bytes(desc, batch, tq, stride, max_kv)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    flag, out = i32([0]), torch.empty_like(dev["q"])
    cf.cf_prefill_attention(desc, dev["q"], i32([b * tq for b in range(batch + 1)]), 0, i32([q_pos] * batch), dev["k_store"], dev["v_store"],
                            n_store, dev["k_self"], dev["v_self"], table, i32([len(x) for x in segs]), stride, batch, tq, max_kv, out,
                            None, None, 1, ws, need, flag)
    # the same call with the segments' masses: the same outputs, bit for bit
    again, mass = torch.empty_like(out), torch.zeros((batch, stride), dtype=torch.float32, device="cuda")
    cf.cf_prefill_attention(desc, dev["q"], i32([b * tq for b in range(batch + 1)]), 0, i32([q_pos] * batch), dev["k_store"], dev["v_store"],
                            n_store, dev["k_self"], dev["v_self"], table, i32([len(x) for x in segs]), stride, batch, tq, max_kv, again,
                            mass, None, 1, ws, need, flag)
    torch.cuda.synchronize()
    assert int(flag.item()) == 0 and torch.equal(again, out)
    got, mass = out.float().cpu().numpy(), mass.cpu().numpy()
    for b in range(batch):
        ks, vs, compact = H.compact_query(segs[b], t["k_store"], t["v_store"])
        part = slice(b * tq, (b + 1) * tq)
        ref, near = H.rounded_key_reference(dtype, t["q"][part], 0, q_pos, ks, vs, t["k_self"], t["v_self"], compact, hkv, 1.0e4)
        assert np.isfinite(got[part]).all()
        assert G.row_error(got[part], ref) <= G.OUT_TOL[dtype]
        assert G.rel_error(mass[b, :len(segs[b])], near) <= G.NEAR_MASS_TOL[dtype]
        assert mass[b].sum() == pytest.approx(hq * tq, rel=1e-5)


@pytest.mark.parametrize("n", [1, 31, 32, 33, 255, 257, 479, 480, 545, 1500])        # one split up to 479, the other kernel at 1500
@pytest.mark.parametrize("hq,hkv,dtype", [(32, 32, "bf16"), (28, 4, "f16"), (16, 1, "bf16")])
def test_one_row_over_a_cache(n, hq, hkv, dtype):
    print(f"decode n={n} {hq}/{hkv} {dtype}", flush=True)
    _check(hq, hkv, 1, [[(0, n, 0, 0)]], n, dtype, n, seed=n)


@pytest.mark.parametrize("layout", ["head", "token"])
@pytest.mark.parametrize("batch,hkv", [(3, 4), (40, 8), (70, 4)])        # 12, 320 and 280 units: several splits, one
def test_unequal_conversations(batch, hkv, layout):
    print(f"decode batch={batch} hkv={hkv} {layout}", flush=True)
    rng = np.random.default_rng(batch)
    lens = rng.integers(1, 900, size=batch)
    off = np.concatenate([[0], np.cumsum(lens)])
    _check(2 * hkv, hkv, 1, [[(int(off[b]), int(lens[b]), 0, 0)] for b in range(batch)], int(off[-1]), "bf16", 1000, seed=batch, layout=layout)


@pytest.mark.parametrize("docs", [1, 2, 63, 64])   # tables of 2 entries (attn_solo_kernel), 3, 64 and 65 (attn_tile_kernel)
@pytest.mark.parametrize("group,tq", [(1, 16), (2, 8), (5, 3), (7, 2)])
def test_moved_documents_and_the_causal_own_block(docs, group, tq):
    print(f"decode docs={docs} group={group} tq={tq}", flush=True)
    rng = np.random.default_rng(docs + tq)
    lens = rng.integers(1, 90, size=docs)
    off = np.concatenate([[0], np.cumsum(lens)])
    # every third document keeps its distance to the query: not moved
    new = [(16 if i % 3 == 1 else int(rng.integers(0, 6000))) for i in range(docs)]
    _check(2 * group, 2, tq, [[(int(off[i]), int(lens[i]), 16, new[i]) for i in range(docs)]] * 2, int(off[-1]), "bf16", 0, seed=docs)


def test_scores_that_rise_move_the_reference():
    """Keys whose scores climb tile after tile: every wavefront's reference moves at almost every tile."""
    n, hkv = 800, 2
    rng = np.random.default_rng(3)
    base = rng.standard_normal((1, hkv, 128)).astype(np.float32)
    q = wl.round_to_dtype(np.repeat(base, 2, axis=1), "bf16")
    ramp = np.linspace(0.0, 5.0, n, dtype=np.float32)[:, None, None]
    k = wl.round_to_dtype(ramp * base + 0.1 * rng.standard_normal((n, hkv, 128)).astype(np.float32), "bf16")
    v = wl.round_to_dtype(rng.standard_normal((n, hkv, 128)).astype(np.float32), "bf16")
    own = [wl.round_to_dtype(rng.standard_normal((1, hkv, 128)).astype(np.float32), "bf16") for _ in range(2)]
    desc = cf.make_desc(2 * hkv, hkv, 128, "bf16", 1.0e4, 8192, cf.CF_ROPE_HALF)
    segs = [orc.Segment(0, n, 0, 0, orc.KIND_DOC, 0), orc.Segment(0, 1, 0, n, orc.KIND_SELF, -1)]
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")
    table = cf.segments_to_device(cf.segments_array([(g.tok_offset, g.len, g.stored_start, g.new_start, g.kind, g.doc) for g in segs]))
    need = cf.cf_prefill_workspace_bytes(desc, 1, 1, 2, n + 1)
    ws, flag = torch.zeros(need, dtype=torch.uint8, device="cuda"), i32([0])
    dq, dk, dv, dks, dvs = (pl.to_device(x, "bf16") for x in (q, k, v, *own))
    out = torch.empty_like(dq)
    cf.cf_prefill_attention(desc, dq, i32([0, 1]), n, i32([n]), dk, dv, n, dks, dvs, table, i32([2]), 2, 1, 1, n + 1, out, None, None, 1, ws,
                            need, flag)
    torch.cuda.synchronize()
    ref, _ = orc.prefill_attention(H.f64(q), n, n, k, v, own[0], own[1], segs, hkv, 1.0e4)
    assert G.row_error(out.float().cpu().numpy(), ref) <= G.OUT_TOL["bf16"]
