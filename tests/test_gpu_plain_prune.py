"""GPU tests of what surrounds the attention outside the 16-bit kernels' shapes: the row-by-row kernel behind tables of more than 256
entries, and a prune step after the fp32-precision kernel (slot partials in double) in each of its forms."""

import pytest
import torch

from oracle import cachefocus_oracle as orc
from paper_2502_11101_amd import binding as cf
from paper_2502_11101_amd import workloads as wl
from tests import gpu_harness as G
from tests.test_gpu_parity import _fused_and_separate, _run_single_layer

pytestmark = pytest.mark.gpu

HALF, INTER = cf.CF_ROPE_HALF, cf.CF_ROPE_INTERLEAVED


def _cfg(name, geometry, docs, lens, batch, tq):
    return wl.scaled(wl.CONFIGS["tiny_f32"], name=name, geometry=geometry, n_store_docs=batch * docs, docs_per_query=docs,
                     batch=batch, doc_len_range=lens, tq=tq, prefix_len=3, doc_stored_start=5, n_planted=1)


@pytest.mark.parametrize("docs", [254, 255])       # 256 entries with prefix and own block: the last table in LDS; 257: row by row
@pytest.mark.parametrize("dtype,pairing,d,hq,hkv,tq", [
    ("f32", HALF, 64, 6, 2, 5),
    ("f32", INTER, 48, 2, 2, 3),
    ("f16", HALF, 96, 4, 2, 2),
    ("f16", INTER, 256, 2, 1, 1),
    ("bf16", INTER, 128, 4, 1, 9),
])
def test_tables_on_both_sides_of_256_entries(dtype, pairing, d, hq, hkv, tq, docs):
    cfg = _cfg(f"entries_{docs + 2}_{dtype}_{d}", wl.Geometry(hq, hkv, d, dtype, 1.0e4, 8192), docs, (1, 9), 2, tq)
    _run_single_layer(cfg, pairing, seed=d + tq, layout="head_padded" if tq % 2 else "token")


@pytest.mark.parametrize("dtype,pairing,d,heads,docs,batch", [
    ("f32", HALF, 64, 5, 20, 3),        # up to 64 entries: one wavefront sums the slots
    ("bf16", INTER, 64, 4, 20, 2),
    ("f32", INTER, 32, 3, 80, 3),       # more: the workgroup does
    ("f16", HALF, 96, 2, 130, 2),
    ("f32", HALF, 64, 60, 100, 2),      # 44 bytes a document and 8 a (kv head, slot of 118): 61 040 of the 61 440 the step has
    ("f32", HALF, 64, 61, 100, 2),      # 61 984: separate kernels
])
def test_prune_step_after_the_fp32_precision_kernel(dtype, pairing, d, heads, docs, batch):
    """One call with the prune step against separate calls: outputs, masses, scores and tables bit for bit; the ranking is the oracle's
    on the accumulated scores, and a query's masses add up to its rows."""
    print(f"prune step {dtype} d={d} heads={heads} docs={docs}", flush=True)
    cfg = _cfg(f"prune_{dtype}_{docs}_{heads}", wl.Geometry(heads, heads, d, dtype, 1.0e4, 8192), docs, (1, 3), batch, 2)
    st = wl.build_structure(cfg, seed=docs)
    keep = docs // 3
    a, b = _fused_and_separate(cfg, st, wl.build_layer(cfg, st, seed=heads), keep, cf.CF_ALLOC_SORT, desc=G.desc_of(cfg, pairing))
    assert a["flags"] == 0 and b["flags"] == 0
    for key in ("out", "mass", "score"):
        assert torch.equal(a[key], b[key]), key
    assert torch.equal(a["keep"][:, :keep], b["keep"][:, :keep]) and torch.equal(a["segs"][:, :keep + 2], b["segs"][:, :keep + 2])
    for q in range(batch):
        ref = orc.prune_topk(b["score"][q].cpu().numpy(), st.doc_lens[st.query_docs[q]], list(range(docs)), keep)
        assert a["keep"][q, :keep].tolist() == ref
        assert float(a["mass"][q, :docs + 2].sum()) == pytest.approx(heads * 2, rel=1e-5)


# many queries of few rows over few tokens go row by row: the largest list that does, the next one, and one query less than many
ROUTES = [("f32", HALF, 16, 1, 32, 64, 65, True), ("f32", HALF, 16, 1, 32, 64, 66, False), ("f32", HALF, 16, 2, 32, 64, 10, True),
          ("f32", HALF, 16, 3, 32, 64, 10, False), ("bf16", INTER, 80, 1, 32, 64, 115, True), ("bf16", INTER, 80, 1, 32, 64, 116, False),
          ("f16", HALF, 144, 2, 32, 64, 35, True), ("bf16", HALF, 16, 1, 32, 63, 20, False)]


@pytest.mark.parametrize("dtype,pairing,d,tq,heads,batch,tokens,by_row", ROUTES)
def test_many_queries_of_few_rows(dtype, pairing, d, tq, heads, batch, tokens, by_row):
    print(f"few rows {dtype} d={d} {batch} x {tq} rows, {heads} heads, {tokens} tokens", flush=True)
    doc = (tokens - tq) // 2
    cfg = wl.scaled(wl.CONFIGS["tiny_f32"], name=f"few_{dtype}_{tokens}", geometry=wl.Geometry(heads, heads, d, dtype, 1.0e4, 8192),
                    n_store_docs=2 * batch, docs_per_query=2, batch=batch, doc_len_range=(doc, doc), tq=tq, prefix_len=tokens - tq - 2 * doc,
                    doc_stored_start=5, n_planted=1)
    desc = G.desc_of(cfg, pairing)
    rows_ws = -(-batch * tq * heads * (4 + 1) * 8 // 256) * 256      # prefix, two documents, own block: a pair per row and entry, and one
    assert (cf.cf_prefill_workspace_bytes(desc, batch, tq, 4, tokens) == rows_ws) == by_row
    _run_single_layer(cfg, pairing, seed=tokens)
