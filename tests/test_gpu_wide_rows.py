"""GPU parity of the attention kernel for many stacked rows: every variant (two and three blocks per wavefront, one and two groups of
wavefronts, table in registers and in LDS, one split and several, CAUSAL; attn_cases) over ragged batches whose short queries leave a group
of wavefronts without a tile; then row counts around the step to another row group, short lists with ragged ends, units
on both sides of 256 and long tables."""

import numpy as np
import pytest
import torch

from paper_2502_11101_amd import binding as cf
from paper_2502_11101_amd import pipeline as pl
from paper_2502_11101_amd import workloads as wl
from tests import attn_cases, plan_probe
from tests import gpu_harness as G
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _run(geo, batch, tq, lens, docs, prefix, seed, layout="head"):
    """Every query attends `docs` documents of the given lengths (rotated from query to query); outputs and masses of a few
    queries against the oracle."""
    rng = np.random.default_rng(seed)
    lens = np.asarray(lens, np.int32)
    off = np.concatenate([[prefix], prefix + np.cumsum(lens)]).astype(np.int64)
    picks = np.stack([np.roll(np.arange(len(lens)), b)[:docs] for b in range(batch)]).astype(np.int32)
    cfg = wl.scaled(wl.CONFIGS["tiny_f32"], name=f"wide_{seed}", geometry=geo, n_store_docs=len(lens), docs_per_query=docs, batch=batch,
                    tq=tq, prefix_len=prefix, doc_stored_start=prefix, n_planted=1)
    st = wl.Structure(lens, off, int(off[-1]), picks, np.zeros((batch, 1), np.int32), 0)
    normal = lambda n, h: wl.round_to_dtype(rng.standard_normal((n, h, 128), dtype=np.float32), geo.dtype)
    t = dict(q=normal(batch * tq, geo.n_q_heads), k_self=normal(batch * tq, geo.n_kv_heads), v_self=normal(batch * tq, geo.n_kv_heads),
             k_store=normal(st.n_store_tokens, geo.n_kv_heads), v_store=normal(st.n_store_tokens, geo.n_kv_heads))
    pb = G.make_batch(cfg, st, layout=layout)
    dev = G.upload_layer(cfg, t, layout=layout)
    out = torch.empty_like(dev["q"])
    pb.allocate_initial()
    pb.workspace.fill_(0xFF)                         # whatever an earlier call left: not read
    pb.attention(dev["q"], dev["k_self"], dev["v_self"], dev["k_store"], dev["v_store"], out)
    torch.cuda.synchronize()
    assert pb.flags() == 0
    got, mass = out.float().cpu().numpy(), pb.mass.cpu().numpy()
    for b in sorted({0, batch // 2, batch - 1}):
        segs, q_start, _ = H.initial_segments(cfg, st, b)
        ks, vs, table = H.compact_query(segs, t["k_store"], t["v_store"])
        rows = slice(b * tq, (b + 1) * tq)
        ref, near = H.rounded_key_reference(geo.dtype, t["q"][rows], 0, q_start, ks, vs, t["k_self"], t["v_self"], table,
                                            geo.n_kv_heads, geo.rope_base)
        assert np.isfinite(got[rows]).all()
        assert G.row_error(got[rows], ref) <= G.OUT_TOL[geo.dtype]
        assert G.rel_error(mass[b, :len(segs)], near) <= G.NEAR_MASS_TOL[geo.dtype]
        assert mass[b, :len(segs)].sum() == pytest.approx(geo.n_q_heads * tq, rel=1e-5)


# tiles of a (query, kv head) whose own block is one tile: none but that one, then one, two, three and four before it
SHORT = [[], [1], [31], [32], [33, 1], [63, 32], [65, 31, 2]]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", attn_cases.WIDE, ids=attn_cases.id_of)
def test_variants(case, dtype):
    """The first query has the longest table; the others have a few tiles for the same splits and groups, fewer rows now and then, or none."""
    print(f"variant {attn_cases.id_of(case)} {dtype}", flush=True)
    c = case
    rng = np.random.default_rng(c.tokens + c.batch + c.group)
    docs, total = c.entries - 1, c.tokens - c.tq
    cuts = np.sort(rng.choice(np.arange(1, total), size=docs - 1, replace=False))
    full = np.diff(np.concatenate([[0], cuts, [total]]))

    def table(lens):
        off = np.concatenate([[0], np.cumsum(lens)])
        # every third document keeps its distance to the query: not moved
        return [(int(off[i]), int(n), 16, 16 if i % 3 == 1 else int(rng.integers(0, 6000))) for i, n in enumerate(lens)]

    short = [x for x in SHORT if len(x) <= docs]
    tables = [table(full)] + [table(short[b % len(short)]) for b in range(1, c.batch)]
    lengths = [c.tq] + [0 if b % 11 == 5 else c.tq // 3 if b % 4 == 3 else c.tq for b in range(1, c.batch)]
    G.check_tables(c.group * c.hkv, c.hkv, c.tq, tables, total, dtype, 0, seed=c.tokens, layout="head" if dtype == "bf16" else "token",
                   lengths=lengths, check=sorted({*range(min(c.batch, 13)), c.batch - 1}))


# The next three: two blocks per wavefront and one group, unless said otherwise.
# stacked rows of a kv head: 65 (five blocks), 128, then two row groups or more: 129, 192, 193, 385, 577
@pytest.mark.parametrize("group,tq", [(5, 13), (4, 32), (3, 43), (6, 32), (1, 193), (7, 55), (1, 577)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_row_counts(group, tq, dtype):
    print(f"rows {group * tq} {dtype}", flush=True)
    _run(wl.Geometry(2 * group, 2, 128, dtype, 1.0e4, 8192), 2, tq, [33, 95, 64, 1, 160], 4, 32, seed=group * tq)


# tiles of a (query, kv head): from one to a dozen, ragged ends of 1, 31, 32
@pytest.mark.parametrize("lens", [[1], [31], [32], [33, 1], [63, 32], [65, 31, 2], [200, 1, 129]])
@pytest.mark.parametrize("batch", [3, 140])          # 6 and 280 units
@pytest.mark.parametrize("prefix", [0, 17])
def test_short_tile_lists(lens, batch, prefix):
    print(f"lens {lens} batch {batch} prefix {prefix}", flush=True)
    _run(wl.Geometry(10, 2, 128, "bf16", 1.0e4, 4096), batch, 16, lens, len(lens), prefix, seed=sum(lens) + batch)


@pytest.mark.parametrize("batch", [128, 129])        # 256 and 258 units, three blocks per wavefront: two groups, one
@pytest.mark.parametrize("layout", ["head", "token"])
def test_units_around_the_compute_units(batch, layout):
    print(f"units {2 * batch} {layout}", flush=True)
    _run(wl.Geometry(12, 2, 128, "f16", 1.0e6, 8192), batch, 30, [70, 130, 100, 41], 3, 8, seed=batch, layout=layout)


@pytest.mark.parametrize("docs", [62, 63, 90])       # 64, 65 and 92 table entries
@pytest.mark.parametrize("batch", [1, 130])
def test_table_in_lds(docs, batch):
    print(f"docs {docs} batch {batch}", flush=True)
    lens = np.random.default_rng(docs).integers(1, 70, size=docs)
    _run(wl.Geometry(14, 2, 128, "bf16", 1.0e4, 8192), batch, 12, lens, docs, 32, seed=docs)


def test_non_finite_values_stay_with_the_rows_that_see_them():
    """An infinite value in a document turns its channel infinite in every row of its kv head — not into NaN by a phase that weighs
    nothing — and leaves every other channel and head alone."""
    geo = wl.Geometry(10, 2, 128, "bf16", 1.0e4, 4096)
    rng = np.random.default_rng(5)
    for lens in ([32], [100, 40]):
        n, tq = int(sum(lens)), 16
        normal = lambda m, h: torch.from_numpy(rng.standard_normal((m, h, 128), dtype=np.float32)).to(torch.bfloat16).cuda()
        q, ks, vs = normal(tq, 10), normal(tq, 2), normal(tq, 2)
        k, v = normal(n, 2), normal(n, 2)
        cfg = wl.scaled(wl.CONFIGS["tiny_f32"], name="wide_inf", geometry=geo, n_store_docs=len(lens), docs_per_query=len(lens), batch=1,
                        tq=tq, prefix_len=0, doc_stored_start=0, n_planted=1)
        off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
        st = wl.Structure(np.asarray(lens, np.int32), off, n, np.arange(len(lens), dtype=np.int32)[None], np.zeros((1, 1), np.int32), 0)
        pb = G.make_batch(cfg, st)
        pb.allocate_initial()
        outs = []
        for bad in (False, True):
            if bad:
                v[7, 1, 90] = float("inf")
            out = torch.empty_like(q)
            pb.attention(q, ks, vs, k, v, out)
            torch.cuda.synchronize()
            outs.append(out.float().cpu().reshape(tq, 2, 5, 128))
        hit = torch.zeros(outs[0].shape, dtype=torch.bool)
        hit[:, 1, :, 90] = True
        assert torch.isposinf(outs[1][hit]).all()
        assert torch.equal(outs[0][~hit], outs[1][~hit])


@pytest.mark.parametrize("batch,nsplit", [(64, 2), (128, 1)])
def test_non_finite_values_with_two_groups(batch, nsplit):
    """The same where one long query gives every query two groups of wavefronts and the short ones leave a group with one tile or none."""
    print(f"infinities, two groups, batch {batch}", flush=True)
    geo, tq, lens = wl.Geometry(10, 2, 128, "bf16", 1.0e4, 4096), 16, np.array([700, 400, 32, 1, 33], np.int32)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(off[-1])
    picks = np.array([[0, 1]] + [[2, 3] if b % 2 else [4, 3] for b in range(1, batch)], np.int32)
    cfg = wl.scaled(wl.CONFIGS["tiny_f32"], name="wide_inf_groups", geometry=geo, n_store_docs=len(lens), docs_per_query=2, batch=batch, tq=tq,
                    prefix_len=0, doc_stored_start=0, n_planted=1)
    pb = G.make_batch(cfg, wl.Structure(lens, off, n, picks, np.zeros((batch, 1), np.int32), 0))
    p = plan_probe.plan(10, 2, batch, tq, pb.seg_stride, pb.max_kv_tokens, pb.ws_bytes)
    assert (p.groups, p.nsplit) == (2, nsplit)
    pb.allocate_initial()
    rng = np.random.default_rng(6)
    normal = lambda m, h: torch.from_numpy(rng.standard_normal((m, h, 128), dtype=np.float32)).to(torch.bfloat16).cuda()
    q, ks, vs, k, v = normal(batch * tq, 10), normal(batch * tq, 2), normal(batch * tq, 2), normal(n, 2), normal(n, 2)
    outs = []
    for bad in (False, True):
        if bad:
            v[350, 0, 5] = float("inf")              # in the middle of the long query's first document
            v[int(off[2]) + 31, 1, 90] = float("inf")        # the last token of the odd queries' first
        out = torch.empty_like(q)
        pb.attention(q, ks, vs, k, v, out)
        torch.cuda.synchronize()
        outs.append(out.float().cpu().reshape(batch, tq, 2, 5, 128))
    hit = torch.zeros(outs[0].shape, dtype=torch.bool)
    hit[0, :, 0, :, 5] = True
    hit[1::2, :, 1, :, 90] = True
    assert torch.isfinite(outs[0]).all() and torch.isposinf(outs[1][hit]).all()
    assert torch.equal(outs[0][~hit], outs[1][~hit])


# rows 65 (five blocks) to 300 (two row groups) of one head, and of several heads, whose blocks hold tokens of all of them
OWN = [(1, 4, 70, 65, 0), (1, 4, 70, 128, 32), (1, 2, 140, 160, 57), (1, 2, 140, 192, 100), (1, 3, 90, 193, 1), (1, 2, 140, 300, 32), (7, 2, 70, 40, 40),
       (6, 3, 60, 33, 16), (2, 2, 140, 97, 33),
       (7, 2, 70, 40, 300), (1, 3, 90, 193, 250)]            # several row groups and a shorter own block


@pytest.mark.parametrize("own_first", [False, True])
@pytest.mark.parametrize("group,hkv,batch,tq,prefix", OWN)
def test_own_block_of_half_the_list(group, hkv, batch, tq, prefix, own_first):
    """Documents encoded over a prefix, in one split: row blocks leave out the tiles past their last row where the own block ends the list (and
    leave out nothing where it does not).  Queries of every length, of none and of one row among them."""
    print(f"own block {group} {hkv} {batch} {tq} {prefix} {own_first}", flush=True)
    p = plan_probe.plan(group * hkv, hkv, batch, tq, 1 + (prefix > 0), prefix + tq)
    assert p.wide == 2                               # CAUSAL
    lengths = [tq, 1, tq - 1, 17, tq // 2, 0, 33 % tq, 64 % tq] + [int(x) for x in np.random.default_rng(tq).integers(1, tq + 1, size=batch - 8)]
    new = 0 if tq % 2 else 500                       # the prefix as it is, or moved
    G.check_tables(group * hkv, hkv, tq, [[(0, prefix, 0, new)] if prefix else []] * batch, max(prefix, 1), "bf16" if tq % 3 else "f16", 0, seed=tq,
                   lengths=lengths, check=[*range(10), batch - 1], own_first=own_first)


@pytest.mark.parametrize("group,hkv,batch,tq,prefix", [(1, 4, 70, 65, 16), (1, 4, 70, 128, 32), (1, 2, 140, 160, 57), (1, 3, 90, 193, 1), (7, 2, 70, 40, 40),
                                                       (6, 3, 60, 33, 16)])
def test_infinities_of_an_own_block_stay_behind_it(group, hkv, batch, tq, prefix):
    """An infinite value at token T of the own block turns its channel infinite in the rows from T on.  The rows of a 16-row block that ends before
    T's tile keep every bit, wherever in the list that tile lies."""
    print(f"own infinity {group} {hkv} {batch} {tq} {prefix}", flush=True)
    p = plan_probe.plan(group * hkv, hkv, batch, tq, 2, prefix + tq)
    assert p.wide == 2                               # CAUSAL
    desc = cf.make_desc(group * hkv, hkv, 128, "bf16", 1.0e4, 8192, cf.CF_ROPE_HALF)
    n = prefix + batch * tq
    gen = torch.Generator(device="cuda").manual_seed(tq)
    normal = lambda rows, heads: torch.randn((rows, heads, 128), generator=gen, device="cuda").to(torch.bfloat16)
    q, k, v, ks, vs = normal(batch * tq, group * hkv), normal(batch * tq, hkv), normal(batch * tq, hkv), normal(n, hkv), normal(n, hkv)
    sb = pl.StoreBuilder(desc, prefix + tq * np.arange(batch), np.full(batch, tq), np.full(batch, prefix), prefix, n)
    bad = [tq - 1 if b % 2 else (5 * b) % tq for b in range(batch)]      # the last token of every other document, any of the others'
    outs = []
    for infinite in (False, True):
        if infinite:
            for b, t in enumerate(bad):
                v[b * tq + t, b % hkv, (5, 90)[b // 2 % 2]] = float("inf")
        out = torch.empty_like(q)
        sb.attend(q, k, v, ks, vs, out)
        torch.cuda.synchronize()
        outs.append(out.float().cpu().reshape(batch, tq, hkv, group, 128))
    assert torch.isfinite(outs[0]).all()
    rows = np.arange(tq * group).reshape(tq, group)
    block_end = torch.from_numpy(np.minimum((rows | 15) // group, tq - 1))       # the last token among a row's block
    for b, t in enumerate(bad):
        h, c = b % hkv, (5, 90)[b // 2 % 2]
        assert torch.isposinf(outs[1][b, t:, h, :, c]).all(), b
        ahead = block_end < t // 32 * 32
        assert torch.equal(outs[1][b, :, h, :, c][ahead], outs[0][b, :, h, :, c][ahead]), b
        hit = torch.zeros(outs[0][b].shape, dtype=torch.bool)
        hit[:, h, :, c] = True
        assert torch.equal(outs[0][b][~hit], outs[1][b][~hit]), b
