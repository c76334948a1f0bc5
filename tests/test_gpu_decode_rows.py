"""GPU parity of the attention kernel for one 16-row block (decode steps): every wavefront streams tiles of its own.
Tile counts from fewer than the wavefronts to fourteen each, ragged ends, several splits and one, moved and unmoved keys, references that
move on the way, rows from one to sixteen with the causal own block, whole layers with their scores and prune events, and the
longer tables that the other kernel keeps."""

import numpy as np
import pytest
import torch

from paper_2502_11101_amd import binding as cf
from paper_2502_11101_amd import workloads as wl
from tests import attn_cases, plan_probe
from tests import gpu_harness as G
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 31, 32, 33, 255, 257, 478, 479, 480, 545, 1500])   # 32 heads: one split up to 478, the other kernel at 1500
@pytest.mark.parametrize("hq,hkv,dtype", [(32, 32, "bf16"), (28, 4, "f16"), (16, 1, "bf16")])
def test_one_row_over_a_cache(n, hq, hkv, dtype):
    print(f"decode n={n} {hq}/{hkv} {dtype}", flush=True)
    G.check_tables(hq, hkv, 1, [[(0, n, 0, 0)]], n, dtype, n, seed=n)


@pytest.mark.parametrize("layout", ["head", "token"])
@pytest.mark.parametrize("batch,hkv", [(3, 4), (40, 8), (70, 4), (64, 16), (65, 16)])      # 12 units: several splits; 320, 280, 1024: one; 1040: the other kernel
def test_unequal_conversations(batch, hkv, layout):
    print(f"decode batch={batch} hkv={hkv} {layout}", flush=True)
    rng = np.random.default_rng(batch)
    lens = rng.integers(1, 900, size=batch)
    off = np.concatenate([[0], np.cumsum(lens)])
    G.check_tables(2 * hkv, hkv, 1, [[(int(off[b]), int(lens[b]), 0, 0)] for b in range(batch)], int(off[-1]), "bf16", 1000, seed=batch, layout=layout)


@pytest.mark.parametrize("docs", [1, 2, 63, 64])   # tables of 2 entries (attn_solo_kernel), 3, 64 and 65 (attn_tile_kernel)
@pytest.mark.parametrize("group,tq", [(1, 16), (2, 8), (5, 3), (7, 2)])
def test_moved_documents_and_the_causal_own_block(docs, group, tq):
    print(f"decode docs={docs} group={group} tq={tq}", flush=True)
    rng = np.random.default_rng(docs + tq)
    lens = rng.integers(1, 90, size=docs)
    off = np.concatenate([[0], np.cumsum(lens)])
    # every third document keeps its distance to the query: not moved
    new = [(16 if i % 3 == 1 else int(rng.integers(0, 6000))) for i in range(docs)]
    G.check_tables(2 * group, 2, tq, [[(int(off[i]), int(lens[i]), 16, new[i]) for i in range(docs)]] * 2, int(off[-1]), "bf16", 0, seed=docs)


@pytest.mark.parametrize("pattern", ["rising", "falling", "saw", "spike", "moved"])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", attn_cases.SOLO, ids=attn_cases.id_of)
def test_long_runs_of_a_wavefront(case, dtype, pattern):
    """Conversations of unequal length over one cache, up to fourteen tiles per wavefront.  `rising` and the others: keys with a growing
    share of the query's direction, so that a wavefront's reference moves again and again and takes what it has summed with it (about ten
    nats over a run of 400 tokens); `moved`: plain keys that are moved."""
    print(f"runs {attn_cases.id_of(case)} {dtype} {pattern}", flush=True)
    rng = np.random.default_rng(case.tokens + case.batch)
    cached = case.tokens - case.tq
    lens = [cached, cached // 2, 1] + [int(x) for x in rng.integers(1, cached + 1, size=case.batch - 3)]

    def shape(t, rng):
        if pattern == "moved":
            return
        i = np.arange(cached)
        share = {"rising": 8.0 * i / cached, "falling": 8.0 - 8.0 * i / cached, "saw": 6.0 * (i % 300) / 300,
                 "spike": np.where(i % 700 == 350, 6.0, 0.0)}[pattern]
        base = rng.standard_normal((1, case.hkv, 128)).astype(np.float32)
        rd = lambda x: wl.round_to_dtype(x.astype(np.float32), dtype)
        t["q"] = rd(np.repeat(base, case.hq // case.hkv, axis=1) + 0.1 * t["q"])
        t["k_store"] = rd(share[:, None, None] * base + 0.1 * t["k_store"])
        t["k_self"] = rd(share.max() * base + 0.1 * t["k_self"])        # as much as the largest, so that no mass vanishes

    new = 900 if pattern == "moved" else 0
    G.check_tables(case.hq, case.hkv, case.tq, [[(0, n, 0, new)] for n in lens], cached, dtype, 0, seed=case.tokens,
                   layout="head" if dtype == "bf16" else "token", check=[0, 1, 2, case.batch - 1], shape=shape)


def _layers_over_one_document(cfg, st, layers, keeps, deferred):
    """A stack whose tables have two entries, a document and the own block."""
    pb = G.make_batch(cfg, st, layout="head")
    assert pb.seg_stride == 3 and cfg.prefix_len == 0
    pb.seg_stride = 2
    pb.segs, pb.next_segs = pb.segs[:, :2].contiguous(), pb.next_segs[:, :2].contiguous()
    pb.mass = pb.mass[:, :2].contiguous()
    pb.ws_bytes = cf.cf_prefill_workspace_bytes(pb.desc, pb.batch, pb.tq, 2, pb.max_kv_tokens)
    pb.workspace = torch.full((pb.ws_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
    g = cfg.geometry
    assert plan_probe.plan(g.n_q_heads, g.n_kv_heads, pb.batch, pb.tq, 2, pb.max_kv_tokens, pb.ws_bytes).groups == 8
    pb.allocate_initial()
    outs, tables = [], []
    for i, dev in enumerate(layers):
        out, args = torch.empty_like(dev["q"]), (dev["q"], dev["k_self"], dev["v_self"], dev["k_store"], dev["v_store"])
        if deferred is None:                         # the separate calls
            pb.attention(*args, out)
            if i in keeps:
                pb.prune(1)
        else:
            pb.layer(*args, out, keep=1 if i in keeps else None, defer=deferred and i not in keeps and i != len(layers) - 1)
        outs.append(out)
        if i in keeps:
            torch.cuda.synchronize()
            tables += [pb.score.clone(), pb.keep_idx.clone(), pb.n_keep.clone(), pb.next_segs.clone(), pb.next_q_start.clone()]
            pb.advance()
    torch.cuda.synchronize()
    assert pb.flags() == 0
    return outs, tables + [pb.score.clone()], pb.mass.clone()


@pytest.mark.parametrize("geo,batch,tq,length", [(wl.Geometry(8, 2, 128, "bf16", 1.0e4, 8192), 3, 4, 700),        # eight splits
                                                 (wl.Geometry(8, 8, 128, "f16", 1.0e4, 8192), 40, 16, 150)])      # one
def test_layers_over_one_document(geo, batch, tq, length):
    """cf_prefill_layer, deferred and not, against the separate calls and its scores against the oracle."""
    print(f"layers over one document, batch {batch}", flush=True)
    n_layers, keeps = 5, (2,)
    cfg = wl.scaled(wl.CONFIGS["tiny_f32"], name=f"one_document_{batch}", geometry=geo, n_store_docs=batch, docs_per_query=1, batch=batch,
                    doc_len_range=(length - 60, length), tq=tq, prefix_len=0, doc_stored_start=8, n_planted=1)
    st = wl.build_structure(cfg, seed=batch)
    tensors = [wl.build_layer(cfg, st, layer, seed=batch + layer) for layer in range(n_layers)]
    layers = [G.upload_layer(cfg, t, "head") for t in tensors]
    apart, eager, lazy = (_layers_over_one_document(cfg, st, layers, keeps, deferred) for deferred in (None, False, True))
    assert all(torch.equal(x, y) for x, y in zip(apart[0], eager[0])) and all(torch.equal(x, y) for x, y in zip(eager[0], lazy[0]))
    assert all(torch.equal(x, y) for x, y in zip(eager[1], lazy[1])) and torch.equal(eager[2], lazy[2])
    assert all(torch.equal(x, y) for x, y in zip(apart[1][1:5], eager[1][1:5]))
    assert G.rel_error(eager[1][0].cpu().numpy(), apart[1][0].cpu().numpy()) < 2e-6        # the same parts, added in another order
    assert G.rel_error(eager[2].cpu().numpy(), apart[2].cpu().numpy()) < 2e-6
    ref = np.zeros((batch, 1))
    for layer in range(keeps[0] + 1):
        t = tensors[layer]
        for b in range(batch):
            segs, q_start, _ = H.initial_segments(cfg, st, b)
            ks, vs, table = H.compact_query(segs, t["k_store"], t["v_store"])
            part = slice(b * tq, (b + 1) * tq)
            out, mass = H.rounded_key_reference(geo.dtype, t["q"][part], 0, q_start, ks, vs, t["k_self"], t["v_self"], table, geo.n_kv_heads,
                                                geo.rope_base)
            ref[b] += H.doc_scores(table, mass, 1)
            assert G.row_error(eager[0][layer][part].float().cpu().numpy(), out) <= G.OUT_TOL[geo.dtype]
    assert G.rel_error(eager[1][0].cpu().numpy(), ref) <= G.NEAR_MASS_TOL[geo.dtype]
