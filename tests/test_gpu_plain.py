"""GPU parity of the attention path that keeps fp32 precision for every type (fp32, head sizes other than 128,
interleaved pairs): the edges of its row blocks, tiles, head paddings and plans, against the oracle."""

import numpy as np
import pytest
import torch

from paper_2502_11101_amd import binding as cf
from paper_2502_11101_amd import pipeline as pl
from paper_2502_11101_amd import workloads as wl
from tests import gpu_harness as G
from tests import helpers as H
from tests.test_gpu_parity import _run_single_layer

pytestmark = pytest.mark.gpu

HALF, INTER = cf.CF_ROPE_HALF, cf.CF_ROPE_INTERLEAVED


def _cfg(name, geometry, docs, lens, batch, tq, prefix):
    return wl.scaled(wl.CONFIGS["tiny_f32"], name=name, geometry=geometry, n_store_docs=batch * docs, docs_per_query=docs,
                     batch=batch, doc_len_range=lens, tq=tq, prefix_len=prefix, doc_stored_start=prefix + 3, n_planted=1)


@pytest.mark.parametrize("dtype,pairing,d,hq,hkv,tq,docs,lens,batch,prefix", [
    ("f32", HALF, 16, 2, 2, 1, 1, (1, 1), 1, 0),           # one row, one token, the smallest head
    ("f32", INTER, 48, 2, 1, 8, 3, (15, 17), 2, 1),        # exactly one row block, lengths round a tile
    ("f32", HALF, 128, 2, 2, 17, 9, (40, 90), 1, 7),       # two row blocks, several splits
    ("f32", HALF, 208, 3, 3, 20, 4, (1, 40), 1, 16),       # padded to 256
    ("f32", INTER, 64, 4, 1, 33, 100, (1, 9), 1, 2),       # nine row blocks in three groups, table in LDS
    ("bf16", INTER, 128, 4, 4, 48, 10, (100, 200), 1, 32), # three row blocks, splits
    ("bf16", HALF, 80, 2, 1, 16, 5, (31, 33), 3, 33),      # tiles of 31 .. 33 tokens
    ("bf16", INTER, 256, 4, 2, 35, 6, (20, 70), 1, 5),
    ("bf16", HALF, 96, 1, 1, 1, 40, (60, 160), 1, 0),      # a decode step's single row over many tokens
    ("f16", HALF, 64, 6, 3, 5, 12, (90, 140), 2, 8),
    ("f16", INTER, 144, 2, 2, 64, 3, (64, 64), 1, 0),      # four full row blocks, full tiles
    ("f16", HALF, 256, 2, 1, 7, 2, (5, 50), 1, 3),
])
def test_plain_path_edges(dtype, pairing, d, hq, hkv, tq, docs, lens, batch, prefix):
    cfg = _cfg(f"plain_{dtype}_{d}_{tq}", wl.Geometry(hq, hkv, d, dtype, 1.0e4, 8192), docs, lens, batch, tq, prefix)
    _run_single_layer(cfg, pairing, seed=d + tq, layout="head_padded" if tq % 2 else "token")


def test_plain_path_query_at_the_top_of_the_fp16_range():
    """Query components near 65504 turn into components past it: they are handled in fp32 all the same."""
    cfg = _cfg("plain_f16_top", wl.Geometry(2, 2, 64, "f16", 1.0e4, 4096), 4, (30, 50), 1, 9, 4)
    st = wl.build_structure(cfg, seed=91)
    t = wl.build_layer(cfg, st, seed=92)
    t["q"] = (np.sign(t["q"]) * np.float32(60000.0)).astype(np.float16)
    for k in ("k_self", "k_store"):
        t[k] = (t[k].astype(np.float32) * 1e-4).astype(np.float16)
    pb = G.make_batch(cfg, st)
    dev = G.upload_layer(cfg, t)
    out = torch.empty_like(dev["q"])
    pb.allocate_initial()
    pb.attention(dev["q"], dev["k_self"], dev["v_self"], dev["k_store"], dev["v_store"], out)
    torch.cuda.synchronize()
    segs, q_start, _ = H.initial_segments(cfg, st, 0)
    ref_out, ref_mass = H.oracle_query(cfg, st, t, 0, segs, q_start)
    assert pb.flags() == 0
    assert G.row_error(out.float().cpu().numpy(), ref_out) <= 2e-3
    assert G.rel_error(pb.mass.cpu().numpy()[0, :len(segs)], ref_mass) <= 1e-4


@pytest.mark.parametrize("tokens", [700, 2000])
@pytest.mark.parametrize("tq", [16, 20, 40])           # one, two and four row blocks: up to 8, 16 and 32 splits to merge
@pytest.mark.parametrize("dtype,pairing,d", [("f32", HALF, 64), ("f32", HALF, 80), ("bf16", INTER, 128), ("f16", HALF, 144)])
def test_merge_of_splits(dtype, pairing, d, tq, tokens):
    """The merge with masses against the oracle, and without them: the same outputs, bit for bit."""
    cfg = _cfg(f"plain_merge_{d}_{tq}_{tokens}", wl.Geometry(2, 2, d, dtype, 1.0e4, 8192), 3, (tokens // 3 - 9, tokens // 3), 1, tq, 5)
    _run_single_layer(cfg, pairing, seed=d + tq, layout="head")
    st = wl.build_structure(cfg, seed=d)
    pb, dev = G.make_batch(cfg, st, pairing), G.upload_layer(cfg, wl.build_layer(cfg, st, seed=tq))
    pb.allocate_initial()
    out, again = torch.empty_like(dev["q"]), torch.empty_like(dev["q"])
    pb.attention(dev["q"], dev["k_self"], dev["v_self"], dev["k_store"], dev["v_store"], out)
    pb.workspace.fill_(0xFF)
    cf.cf_prefill_attention(pb.desc, dev["q"], pb.q_off, pb.q_stored_start, pb.q_start, dev["k_store"], dev["v_store"], st.n_store_tokens,
                            dev["k_self"], dev["v_self"], pb.segs, pb.n_seg, pb.seg_stride, 1, tq, pb.max_kv_tokens, again, None, None, 1,
                            pb.workspace, pb.ws_bytes, pb.dev_flag)
    torch.cuda.synchronize()
    assert pb.flags() == 0 and torch.isfinite(again).all() and torch.equal(out, again)


@pytest.mark.parametrize("dtype,pairing,d,docs", [("bf16", INTER, 128, 5), ("f32", HALF, 64, 4), ("f32", HALF, 64, 14), ("f16", INTER, 128, 5)])
def test_eight_splits_or_more(dtype, pairing, d, docs):
    """32 units on both sides of four tiles a group, where all but fp16 keep to eight splits."""
    cfg = _cfg(f"plain_eight_{dtype}_{docs}", wl.Geometry(32, 32, d, dtype, 1.0e4, 8192), docs, (80, 100), 1, 40, 9)
    _run_single_layer(cfg, pairing, seed=d + docs, layout="head")
