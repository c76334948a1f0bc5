"""Values on the attention path outside the 16-bit kernels' shapes, on tables made by hand: what must come out exactly, and what
must not be lost."""

import numpy as np
import pytest
import torch

from paper_2502_11101_amd import binding as cf
from paper_2502_11101_amd import pipeline as pl
from paper_2502_11101_amd import workloads as wl
from tests import gpu_harness as G
from tests import helpers as H

pytestmark = pytest.mark.gpu

HALF, INTER = cf.CF_ROPE_HALF, cf.CF_ROPE_INTERLEAVED
I32 = dict(dtype=torch.int32, device="cuda")
D = 64


def _attend(dtype, q, ks, vs, lens, own=None, tq=1):
    """Every query attends the first sum(lens) tokens of the store as segments of these lengths, nothing moved, then its own block
    (keys, values) if there is one.  One head of D channels.  Returns outputs and masses."""
    batch = q.shape[0] // tq
    n_seg = len(lens) + (own is not None)
    off = np.concatenate([[0], np.cumsum(lens)])
    tables = []
    for b in range(batch):
        tables += [(int(off[i]), int(l), 0, 0, cf.CF_SEG_DOC, i) for i, l in enumerate(lens)]
        if own is not None:
            tables.append((b * tq, tq, 0, 0, cf.CF_SEG_SELF, -1))
    desc = cf.make_desc(1, 1, D, dtype, 1.0e4, 8192, INTER)
    dev = [pl.to_device(np.ascontiguousarray(x), dtype) if x is not None else None for x in (q, ks, vs, *(own or (None, None)))]
    kv = int(off[-1]) + (tq if own is not None else 0)
    ws_bytes = cf.cf_prefill_workspace_bytes(desc, batch, tq, n_seg, kv)
    ws = torch.full((ws_bytes,), 0xFF, dtype=torch.uint8, device="cuda")
    out, mass = torch.full_like(dev[0], 7.0), torch.full((batch, n_seg), -1.0, device="cuda")
    flag = torch.zeros(1, **I32)
    cf.cf_prefill_attention(desc, dev[0], torch.arange(0, (batch + 1) * tq, tq, **I32), 0, torch.zeros(batch, **I32), dev[1], dev[2],
                            ks.shape[0], dev[3], dev[4], cf.segments_to_device(cf.segments_array(tables)),
                            torch.full((batch,), n_seg, **I32), n_seg, batch, tq, kv, out, mass, None, 0, ws, ws_bytes, flag)
    torch.cuda.synchronize()
    assert flag.item() == 0
    return out.float().cpu().numpy(), mass.cpu().numpy()


@pytest.mark.parametrize("far", [0, 700])          # without and with splits to merge
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_the_mass_of_all_a_row_sees_is_one(dtype, far):
    """13 tokens in one tile have the whole weight of the row: sum over sum, which a division gives as exactly 1 (a product with the
    rounded reciprocal misses it by 2^-24 in some rows).  The other tokens' weights are below the smallest fp32 number."""
    rng = np.random.default_rng(13)
    print(f"mass {dtype} far={far}", flush=True)
    q, ks, vs = (rng.standard_normal((n, 1, D), dtype=np.float32) for n in (64, 13 + far, 13 + far))
    q[:, :, 0], ks[:13, :, 0], ks[13:, :, 0] = 8.0, 0.0, -1000.0
    _, mass = _attend(dtype, q, ks, vs, [13, far] if far else [13])
    assert np.array_equal(mass[:, 0], np.ones(64, np.float32))
    assert np.all(mass[:, 1:] == 0.0)


@pytest.mark.parametrize("small", [20, 28, 33, 36])
@pytest.mark.parametrize("far", [0, 700])          # without and with splits to merge
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
def test_small_probabilities_keep_their_bits(dtype, far, small):
    """A token with 2^-small of the largest probability carries the only values there are: the outputs are its products alone,
    and as exact as the type they are stored in."""
    print(f"small {dtype} far={far} 2^-{small}", flush=True)
    n, tokens = 16, 13 + far
    q, ks, vs = np.zeros((n, 1, D), np.float32), np.zeros((tokens, 1, D), np.float32), np.zeros((tokens, 1, D), np.float32)
    q[:, 0, 0] = 1.0 + np.arange(n) / 128.0         # exact in every type
    ks[5, 0, 0] = -np.float32(np.round(small * np.log(2.0) * np.sqrt(D)))
    ks[13:, 0, 0] = -1200.0
    vs[5] = np.where(np.arange(D) % 2, 1.0, -1.5) * 2.0 ** 15
    out, _ = _attend(dtype, q, ks, vs, [13, far] if far else [13])
    s = np.float64(q[:, 0, 0])[:, None] * np.float64(ks[:, 0, 0])[None] / np.sqrt(D)
    p = np.exp(s - s.max(axis=1, keepdims=True))
    ref = (p / p.sum(axis=1, keepdims=True)) @ np.float64(vs[:, 0])
    # scores up to 2^40 apart in fp32 (two roundings of a number below 64), and one rounding of the result (fp16: to multiples of 2^-24
    # below 2^-14)
    bound = np.abs(ref) * ({"f32": 0.0, "bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype] + 64 * 2.0 ** -23) + (2.0 ** -25 if dtype == "f16" else 0.0)
    assert np.all(np.abs(out[:, 0] - ref) <= bound)


def _reference(q, ks, vs, own, tq):
    """The same in 64 bits: a row's products with the tokens it sees, and no others.  Outputs, and masses of the store and the own block."""
    out, mass = np.zeros((len(q), D)), np.zeros((len(q) // tq, 2))
    for row in range(len(q)):
        b, t = divmod(row, tq)
        k, v = (np.concatenate([x[:, 0], y[b * tq:b * tq + t + 1, 0]]).astype(np.float64) for x, y in ((ks, own[0]), (vs, own[1])))
        with np.errstate(invalid="ignore", over="ignore"):
            s = (k * q[row, 0].astype(np.float64)).sum(axis=1) / np.sqrt(D)
            p = np.exp(s - s.max())
            p /= p.sum()
            out[row] = (p[:, None] * v).sum(axis=0)
        mass[b] += [p[:len(ks)].sum(), p[len(ks):].sum()]
    return out, mass


@pytest.mark.parametrize("store", [9, 700])        # without and with splits to merge
@pytest.mark.parametrize("tq", [3, 20, 60])        # one, two and four row blocks
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("what", ["own value NaN", "own value Inf", "own key NaN", "value Inf", "value NaN", "key weight zero"])
def test_infinities_and_nan_reach_the_rows_that_see_them(what, dtype, tq, store):
    """A row's result does not depend on tokens it does not see, whatever they hold; an infinite value it sees gives an infinite
    channel and a NaN a NaN one; a key whose score is minus infinity has no weight."""
    print(f"non-finite {what}: {dtype} tq={tq} store={store}", flush=True)
    rng = np.random.default_rng(tq + store)
    rows = 2 * tq
    normal = lambda n: torch.from_numpy(rng.standard_normal((n, 1, D), dtype=np.float32)).to(pl.TORCH_DTYPE[dtype]).float().numpy()
    q, k1, v1, ks, vs = normal(rows), normal(rows), normal(rows), normal(store), normal(store)
    at = tq + tq // 2                              # a token of the second query's own block
    if what == "own value NaN": v1[at, 0, 5] = np.nan
    elif what == "own value Inf": v1[at, 0, 62] = -np.inf
    elif what == "own key NaN": k1[at, 0, 7] = np.nan
    elif what == "value Inf": vs[4, 0, 1:4] = np.inf
    elif what == "value NaN": vs[store - 1, 0, 33] = np.nan
    else: q[:, 0, 9], ks[2, 0, 9] = 2.0, -np.inf
    out, mass = _attend(dtype, q, ks, vs, [store], (k1, v1), tq)
    ref, ref_mass = _reference(q, ks, vs, (k1, v1), tq)
    out = out[:, 0].astype(np.float64)
    for kind in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(kind(out), kind(ref))
    ok = np.isfinite(ref)
    assert np.all(np.abs(out[ok] - ref[ok]) <= {"f32": 1e-5, "bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype] * np.maximum(np.abs(ref[ok]), 1e-2) + 1e-5)
    seen = np.isfinite(ref_mass).all(axis=1)       # (a row that sees a NaN key has no masses)
    assert np.allclose(mass[seen], ref_mass[seen], rtol=1e-5)


@pytest.mark.parametrize("dtype,pairing,d,hq,hkv,tq,docs,lens,layout", [
    ("f32", HALF, 208, 4, 2, 11, 6, (20, 90), "head_padded"),      # padded to 256; several splits
    ("bf16", INTER, 256, 2, 1, 35, 4, (20, 70), "token"),          # four row blocks
    ("f16", HALF, 80, 6, 3, 3, 5, (31, 33), "head"),
    ("f32", INTER, 64, 2, 1, 33, 100, (1, 9), "token"),            # table in LDS, two row groups
    ("bf16", INTER, 128, 2, 2, 1, 40, (60, 160), "head_padded"),   # a single row
])
def test_rows_with_an_infinite_value_keep_their_other_channels(dtype, pairing, d, hq, hkv, tq, docs, lens, layout):
    """One infinite value in a re-positioned document: its channel is infinite in every row of the query heads on that kv head, all
    else is as without it, against the oracle."""
    print(f"infinite channel: {dtype} d={d} tq={tq}", flush=True)
    cfg = wl.scaled(wl.CONFIGS["tiny_f32"], name=f"inf_{dtype}_{d}", geometry=wl.Geometry(hq, hkv, d, dtype, 1.0e4, 8192),
                    n_store_docs=docs, docs_per_query=docs, batch=1, doc_len_range=lens, tq=tq, prefix_len=4, doc_stored_start=7, n_planted=1)
    st = wl.build_structure(cfg, seed=d)
    t = wl.build_layer(cfg, st, seed=d + 1)
    segs, q_start, _ = H.initial_segments(cfg, st, 0)
    ref_out, ref_mass = H.oracle_query(cfg, st, t, 0, segs, q_start, pairing="half" if pairing == HALF else "interleaved")
    at = next(s for s in segs if s.kind == cf.CF_SEG_DOC).tok_offset
    t["v_store"] = np.array(t["v_store"])
    t["v_store"][at, hkv - 1, 3] = np.inf
    pb = G.make_batch(cfg, st, pairing, layout)
    dev = G.upload_layer(cfg, t, layout)
    out = torch.empty_like(dev["q"])
    pb.allocate_initial()
    pb.workspace.fill_(0xFF)
    pb.attention(dev["q"], dev["k_self"], dev["v_self"], dev["k_store"], dev["v_store"], out)
    torch.cuda.synchronize()
    assert pb.flags() == 0
    got = out.float().cpu().numpy()
    hit = np.zeros(got.shape, bool)
    hit[:, (hkv - 1) * (hq // hkv):, 3] = True
    assert np.all(np.isposinf(got[hit]))
    assert G.row_error(np.where(hit, 0.0, got), np.where(hit, 0.0, ref_out)) <= G.OUT_TOL[dtype]
    assert G.rel_error(pb.mass.cpu().numpy()[0, :len(segs)], ref_mass) <= 1e-5
