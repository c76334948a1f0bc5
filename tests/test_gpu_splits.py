"""GPU parity of the 16-bit attention path where the number of (query, kv head) units does not divide the 256 compute units:
batches on both sides of the points where a call goes from three splits to two and from two to one."""

import numpy as np
import pytest
import torch

from paper_2502_11101_amd import workloads as wl
from tests import gpu_harness as G
from tests import helpers as H
from tests import plan_probe
from tests.test_gpu_parity import _run_single_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,hkv", [(17, 5), (43, 2), (16, 8), (43, 3), (15, 17)])     # 85, 86, 128, 129, 255 units
def test_split_counts(batch, hkv):
    cfg = wl.scaled(wl.CONFIGS["tiny_f32"], name=f"splits_{batch * hkv}", geometry=wl.Geometry(2 * hkv, hkv, 128, "bf16", 1.0e4, 8192),
                    n_store_docs=batch * 2, docs_per_query=2, batch=batch, doc_len_range=(90, 200), tq=24, prefix_len=32,
                    doc_stored_start=32, n_planted=1)
    # few rows and tokens: the plain oracle's masses to the bound of the other edge shapes, the rounded-key reference's tight
    _run_single_layer(cfg, seed=batch, mass_tol=2e-3, layout="head")


@pytest.mark.parametrize("even", [True, False])
@pytest.mark.parametrize("batch,hkv", [(43, 3), (36, 4), (191, 1)])     # 129, 144, 191 units
def test_two_halves_of_a_long_batch(batch, hkv, even):
    """Single query rows over two of eight long documents each (more than 128 estimated tiles): two splits a query where one would
    leave over a quarter of the compute units idle, at equal lengths and at lengths up to seven times apart."""
    print(f"halves units={batch * hkv} even={even}", flush=True)
    rng = np.random.default_rng(batch)
    lens = np.full(8, 2100, np.int32) if even else np.concatenate([[2200, 2100], rng.integers(300, 2200, size=6)]).astype(np.int32)
    off = np.concatenate([[16], 16 + np.cumsum(lens)]).astype(np.int64)
    picks = np.stack([rng.permutation(8)[:2] for _ in range(batch)]).astype(np.int32)
    picks[batch // 2] = [1, 0]
    cfg = wl.scaled(wl.CONFIGS["tiny_f32"], name=f"halves_{batch * hkv}", geometry=wl.Geometry(hkv, hkv, 128, "bf16", 1.0e4, 8192),
                    n_store_docs=8, docs_per_query=2, batch=batch, tq=1, prefix_len=16, doc_stored_start=16, n_planted=1)
    st = wl.Structure(lens, off, int(off[-1]), picks, np.zeros((batch, 1), np.int32), 0)
    normal = lambda n: wl.round_to_dtype(rng.standard_normal((n, hkv, 128), dtype=np.float32), "bf16")
    t = dict(q=normal(batch), k_self=normal(batch), v_self=normal(batch), k_store=normal(st.n_store_tokens), v_store=normal(st.n_store_tokens))
    pb = G.make_batch(cfg, st)
    assert pb.max_kv_tokens > 128 * 32
    dev = G.upload_layer(cfg, t)
    out = torch.empty_like(dev["q"])
    pb.allocate_initial()
    pb.workspace.fill_(0xFF)
    pb.attention(dev["q"], dev["k_self"], dev["v_self"], dev["k_store"], dev["v_store"], out)
    torch.cuda.synchronize()
    assert pb.flags() == 0
    out_np, mass = out.float().cpu().numpy(), pb.mass.cpu().numpy()
    for b in range(0, batch, 1 + batch // 30):
        segs, q_start, _ = H.initial_segments(cfg, st, b)
        ks, vs, table = H.compact_query(segs, t["k_store"], t["v_store"])
        ref, near = H.rounded_key_reference("bf16", t["q"][b:b + 1], 0, q_start, ks, vs, t["k_self"], t["v_self"], table, hkv, 1.0e4)
        assert G.row_error(out_np[b:b + 1], ref) <= G.OUT_TOL["bf16"]
        assert G.rel_error(mass[b, :len(segs)], near) <= G.NEAR_MASS_TOL["bf16"]
        assert mass[b, :len(segs)].sum() == pytest.approx(hkv, rel=1e-5)


@pytest.mark.parametrize("tokens,nsplit", [(1000, 8), (1120, 9), (2016, 16), (2130, 17), (4200, 32)])
@pytest.mark.parametrize("rows", [16, 17, 32, 33, 64])     # one, two, three and four row blocks: 4, 2 and 1 channel blocks a merging workgroup
def test_merge_of_splits(rows, tokens, nsplit):
    """Every split count on either side of what the merge kernel holds at a time, with masses and without."""
    print(f"merge rows={rows} splits={nsplit}", flush=True)
    assert plan_probe.plan(1, 1, 1, rows, 2, tokens + rows).nsplit == nsplit
    G.check_tables(1, 1, rows, [[(0, tokens, 0, 300)]], tokens, "bf16" if rows & 1 else "f16", 500, seed=rows + nsplit)
