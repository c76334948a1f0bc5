"""The work a program does with this library, as cases that can be timed and compared.

A retrieval-augmented server built on the cached-KV prefill path calls it in six ways, one `kind` each:

  layer       one transformer layer of a batch of queries with its prune event (PrefillBatch.layer)
  stack       a query's whole prefill: initial allocation, every layer, prune events on the way (PrefillBatch)
  decode      one new token per query over its assembled cache, outputs only (cf_prefill_attention)
  encode      documents encoded offline and written to the cache store (StoreBuilder.attend, .write)
  assemble    the survivors of one layer gathered into a contiguous decode cache (cf_assemble_cache)
  reposition  the cached keys of one layer moved to new positions out of place (cf_reposition_keys)

Sizes are those of workloads.CONFIGS, of bench.py and of the ranges the tests cover.  Inputs are seeded Gaussians of
those shapes; the documents of a query are given graded relevance (their keys carry a share of the query's mean
direction), so that a ranking by attention mass has well separated scores, as retrieved passages have.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2502_11101_amd import binding as cf
from paper_2502_11101_amd import pipeline as pl

TORCH = pl.TORCH_DTYPE
SIZE = {"f32": 4, "bf16": 2, "f16": 2}

# head geometries of workloads.CONFIGS: query heads, kv heads, head_dim, rope base, positions
LLAMA2_7B = dict(hq=32, hkv=32, d=128, base=1.0e4, positions=4096)
QWEN2_7B = dict(hq=28, hkv=4, d=128, base=1.0e6, positions=32768)
QWEN2_1P5B = dict(hq=12, hkv=2, d=128, base=1.0e6, positions=32768)
TINY = dict(hq=4, hkv=4, d=64, base=1.0e4, positions=4096)


def listed():
    return [
        # one new token of one conversation over the five surviving passages: the smallest call, made once per layer and token
        dict(name="decode_one", kind="decode", **LLAMA2_7B, dtype="bf16", batch=1, lo=881, hi=881),
        # continuous batching: 32 conversations of unequal length, grouped-query heads
        dict(name="decode_batch", kind="decode", **QWEN2_7B, dtype="bf16", batch=32, lo=1000, hi=5000),
        # the exactness configuration: fp32, head_dim 64 (a reference run)
        dict(name="layer_tiny_f32", kind="layer", **TINY, dtype="f32", pairing="half", layout="token", batch=1, prefix=4,
             docs=4, lo=32, hi=32, tq=8, keep=2, spare=0, strategy="sort"),
        # interactive question answering over ten passages, multi-head attention
        dict(name="layer_llama2_7b", kind="layer", **LLAMA2_7B, dtype="bf16", pairing="half", layout="head", batch=1, prefix=32,
             docs=10, lo=160, hi=160, tq=48, keep=5, spare=0, strategy="sort"),
        # the same under load: eight queries at once, each with passages of its own
        dict(name="layer_llama2_7b_b8", kind="layer", **LLAMA2_7B, dtype="bf16", pairing="half", layout="head", batch=8, prefix=32,
             docs=10, lo=160, hi=160, tq=48, keep=5, spare=0, strategy="sort"),
        # a long context: fifty passages, grouped-query heads
        dict(name="layer_qwen2_7b", kind="layer", **QWEN2_7B, dtype="bf16", pairing="half", layout="head", batch=1, prefix=32,
             docs=50, lo=100, hi=200, tq=64, keep=20, spare=0, strategy="sort"),
        # throughput serving: 64 queries over a store of 10 000 passages, fp16
        dict(name="layer_qwen2_1p5b_b64", kind="layer", **QWEN2_1P5B, dtype="f16", pairing="half", layout="head", batch=64, prefix=0,
             docs=20, lo=100, hi=200, tq=64, keep=8, spare=8720, strategy="sort"),
        # a model that keeps its keys in interleaved pairs, token-major store
        dict(name="layer_interleaved", kind="layer", **LLAMA2_7B, dtype="bf16", pairing="interleaved", layout="token", batch=1,
             prefix=32, docs=10, lo=100, hi=200, tq=48, keep=5, spare=0, strategy="align"),
        # a query's whole prefill: 32 layers, 30 passages, prune events after layers 8, 16, 24 and 32
        dict(name="stack_llama2_7b", kind="stack", **LLAMA2_7B, dtype="bf16", pairing="half", layout="head", batch=1, prefix=32,
             docs=30, lo=160, hi=160, tq=48, layers=32, every=8, spare=0, strategy="sort"),
        # offline: thirty passages encoded for one layer and written to the store
        dict(name="encode_llama2_7b", kind="encode", **LLAMA2_7B, dtype="bf16", layout="head", prefix=32, docs=30, lo=160, hi=160),
        # Alg. 2 Phase 2 without pruning: thirty passages of one layer into a decode cache
        dict(name="assemble_llama2_7b", kind="assemble", **LLAMA2_7B, dtype="bf16", pairing="half", layout="head", batch=1,
             prefix=32, docs=30, lo=160, hi=160, tq=48),
        # the re-positioning pass on its own
        dict(name="reposition_llama2_7b", kind="reposition", **LLAMA2_7B, dtype="bf16", pairing="half", layout="head", docs=30,
             lo=160, hi=160),
    ]


def draw(rng):
    """One more case: a kind and a geometry, sizes log-uniform over their ranges, no more work than the largest listed
    case of its kind."""
    def log_int(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    def lengths(lo, hi):
        a = log_int(lo, hi)
        return dict(lo=a, hi=a if rng.random() < 0.3 else min(2 * hi, int(a * rng.uniform(1.1, 2.0)) + 1))

    kind = rng.choice(["layer", "layer", "layer", "plain_layer", "plain_layer", "stack", "decode", "decode", "encode", "encode",
                       "assemble", "reposition"])
    limit = {k: max(work(c)["bytes"] + work(c)["flops"] / 300 for c in listed() if _group(c) == k)
             for k in {_group(c) for c in listed()}}
    while True:
        geo = dict(rng.choice([LLAMA2_7B, QWEN2_7B, QWEN2_1P5B]))
        dtype = rng.choice(["bf16", "bf16", "f16"])
        if kind in ("layer", "plain_layer"):
            pairing = "half"
            if kind == "plain_layer":           # fp32, interleaved pairs, other head sizes
                geo = dict(rng.choice([TINY, LLAMA2_7B, QWEN2_1P5B]))
                dtype = rng.choice(["f32", "f32", "bf16", "f16"])
                geo["d"] = rng.choice([64, 64, 96, 128, 256])
                pairing = rng.choice(["half", "interleaved"]) if dtype == "f32" or geo["d"] != 128 else "interleaved"
            docs = log_int(3, 56)
            c = dict(kind="layer", **geo, dtype=dtype, pairing=pairing, layout=rng.choice(["head", "token"]),
                     batch=log_int(1, 64), prefix=rng.choice([0, 4, 32, 32, 57]), docs=docs, **lengths(24, 260), tq=log_int(5, 130),
                     keep=max(1, math.ceil(rng.uniform(0.3, 0.7) * docs)), spare=rng.choice([0, 0, 100]),
                     strategy=rng.choice(["sort", "sort", "align"]))
        elif kind == "stack":
            every = rng.choice([2, 4, 7, 8])
            c = dict(kind="stack", **geo, dtype=dtype, pairing="half", layout=rng.choice(["head", "head", "token"]), batch=log_int(1, 4),
                     prefix=32, docs=log_int(8, 50), **lengths(60, 200), tq=log_int(12, 100), layers=every * rng.randint(1, 4),
                     every=every, spare=0, strategy=rng.choice(["sort", "align"]))
        elif kind == "decode":
            c = dict(kind="decode", **geo, dtype=dtype, batch=log_int(1, 64), **lengths(200, 2500))
        elif kind == "encode":
            c = dict(kind="encode", **geo, dtype=dtype, layout=rng.choice(["head", "token"]), prefix=rng.choice([0, 32, 57]),
                     docs=log_int(1, 300), **lengths(40, 300))
        elif kind == "assemble":
            c = dict(kind="assemble", **geo, dtype=dtype, pairing=rng.choice(["half", "half", "interleaved"]),
                     layout=rng.choice(["head", "token"]), batch=log_int(1, 32), prefix=32, docs=log_int(3, 50), **lengths(60, 200),
                     tq=log_int(8, 100))
        else:
            c = dict(kind="reposition", **geo, dtype=rng.choice([dtype, "f32"]), pairing=rng.choice(["half", "half", "interleaved"]),
                     layout=rng.choice(["head", "token"]), docs=log_int(3, 300), **lengths(40, 200))
        # a document must fit the positional range, and the groups of a query with it
        if c["hi"] + c.get("tq", 1) + c.get("prefix", 0) >= c["positions"]:
            continue
        w = work(c)
        if w["bytes"] + w["flops"] / 300 <= limit[_group(c)]:
            return c


def _group(c):
    """Kinds whose cost is compared: the layers outside bf16 / fp16, head_dim 128, half-split pairs stand on their own."""
    if c["kind"] == "layer":
        return "layer" if c["dtype"] != "f32" and c["d"] == 128 and c["pairing"] == "half" else "plain_layer"
    return c["kind"]


# ------------------------------------------------------------------------------------------------ structure
def _lens(c, n, seed):
    return np.random.default_rng(seed).integers(c["lo"], c["hi"] + 1, size=n, dtype=np.int64)


def _alive(c):
    """Documents per layer of a stack: every `every` layers 60 % are kept."""
    alive, keeps, k = [], {}, c["docs"]
    for layer in range(c["layers"]):
        alive.append(k)
        if (layer + 1) % c["every"] == 0:
            k = max(1, math.ceil(0.6 * k))
            keeps[layer] = k
    return alive, keeps


def work(case):
    """Keys, values, queries and outputs once each; 4 * d flops per (query head, row, visible key)."""
    c, e = case, SIZE[case["dtype"]]
    mean = 0.5 * (c["lo"] + c["hi"])
    row_kv = 2 * c["hkv"] * c["d"] * e          # K and V of one token
    row_q = 2 * c["hq"] * c["d"] * e            # q and out of one row
    per_pair = 4.0 * c["d"] * c["hq"]
    kind = c["kind"]
    if kind in ("layer", "stack"):
        alive = [c["docs"]] if kind == "layer" else _alive(c)[0]
        tq, b = c["tq"], c["batch"]
        own = tq * (tq + 1) / 2
        tokens = sum(c["prefix"] + n * mean + tq for n in alive) * b
        pairs = sum((c["prefix"] + n * mean) * tq + own for n in alive) * b
        return {"bytes": tokens * row_kv + len(alive) * b * tq * row_q, "flops": pairs * per_pair}
    if kind == "decode":
        return {"bytes": c["batch"] * ((mean + 1) * row_kv + row_q), "flops": c["batch"] * (mean + 1) * per_pair}
    if kind == "encode":                        # q, k, v read, out written; k, v read and written to the store
        n = c["docs"] * mean
        return {"bytes": n * row_q + 2 * n * row_kv + c["prefix"] * row_kv,
                "flops": c["docs"] * (mean * c["prefix"] + mean * (mean + 1) / 2) * per_pair}
    if kind == "assemble":
        n = c["batch"] * (c["prefix"] + c["docs"] * mean + c["tq"])
        return {"bytes": 2 * n * row_kv, "flops": n * 3.0 * c["hkv"] * c["d"]}
    n = c["docs"] * mean                        # reposition: keys only
    return {"bytes": n * row_kv, "flops": n * 3.0 * c["hkv"] * c["d"]}


def tolerance(case):
    if case["kind"] in ("assemble", "reposition"):          # one rotation, one rounding; values are copied
        return {"rel": {"f32": 1e-6, "bf16": 1e-3, "f16": 2e-4}[case["dtype"]],
                "max": {"f32": 1e-5, "bf16": 1.6e-2, "f16": 2e-3}[case["dtype"]]}
    if _group(case) == "plain_layer":                       # fp32 throughout, the outputs rounded once
        return {"rel": {"f32": 1e-5, "bf16": 4e-3, "f16": 1e-3}[case["dtype"]]}
    return {"rel": {"bf16": 1e-2, "f16": 2e-3}[case["dtype"]]}


# ------------------------------------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)


def _normal(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(TORCH[dtype])


def _desc(c, n_store_tokens):
    ts, hs = (0, 0) if c.get("layout", "head") == "token" else pl.store_strides(n_store_tokens, c["hkv"], c["d"], "head")
    pairing = cf.CF_ROPE_INTERLEAVED if c.get("pairing") == "interleaved" else cf.CF_ROPE_HALF
    return cf.make_desc(c["hq"], c["hkv"], c["d"], c["dtype"], c["base"], c["positions"], pairing,
                        store_token_stride=ts, store_head_stride=hs)


def _store_shape(c, n_tokens):
    return (n_tokens, c["hkv"], c["d"]) if c.get("layout", "head") == "token" else (c["hkv"], n_tokens, c["d"])


class _Tables:
    """Which documents each query has, where they lie in the store, and the batch's device tables."""

    def __init__(self, c, seed):
        b, k = c["batch"], c["docs"]
        rng = np.random.default_rng(seed)
        n_docs = b * k + c.get("spare", 0)
        lens = _lens(c, n_docs, seed + 1)
        off = c["prefix"] + np.concatenate([[0], np.cumsum(lens)])
        self.n_tokens = int(off[-1])
        pick = rng.permutation(n_docs)[:b * k].reshape(b, k)
        self.doc_len, self.doc_off = lens[pick], off[:-1][pick]
        self.desc = _desc(c, self.n_tokens)
        self.pb = pl.PrefillBatch(self.desc, self.doc_off, self.doc_len, c["tq"], c["prefix"], c["prefix"], self.n_tokens)
        # the tokens of the queries' documents: store index, owning query, relevance of their document
        gains = np.stack([rng.permutation(np.linspace(0.0, 0.6, k)) for _ in range(b)])
        flat_len, flat_off = self.doc_len.reshape(-1), self.doc_off.reshape(-1)
        starts = np.concatenate([[0], np.cumsum(flat_len)])[:-1]
        within = np.arange(int(flat_len.sum())) - np.repeat(starts, flat_len)
        self.tok = torch.from_numpy(np.repeat(flat_off, flat_len) + within).cuda()
        self.owner = torch.from_numpy(np.repeat(np.repeat(np.arange(b), k), flat_len)).cuda()
        self.gain = torch.from_numpy(np.repeat(gains.reshape(-1), flat_len).astype(np.float32)).cuda()

    def layer(self, c, gen):
        b, tq, hkv, d, dt = c["batch"], c["tq"], c["hkv"], c["d"], c["dtype"]
        q = _normal(gen, (b * tq, c["hq"], d), dt)
        own = [_normal(gen, (b * tq, hkv, d), dt) for _ in range(2)]
        store = [_normal(gen, _store_shape(c, self.n_tokens), dt) for _ in range(2)]
        mean = q.float().reshape(b, tq, hkv, c["hq"] // hkv, d).mean(dim=(1, 3))
        mean = mean / mean.square().mean(dim=-1, keepdim=True).sqrt()
        keys = store[0] if c["layout"] == "token" else store[0].transpose(0, 1)        # [token][kv head][d]
        for at in range(0, len(self.tok), 1 << 16):
            t, o, g = (x[at:at + (1 << 16)] for x in (self.tok, self.owner, self.gain))
            keys[t] = (keys[t].float() + g[:, None, None] * mean[o]).to(keys.dtype)
        return dict(q=q, k_self=own[0], v_self=own[1], k_store=store[0], v_store=store[1])


STRATEGY = {"sort": cf.CF_ALLOC_SORT, "align": cf.CF_ALLOC_ALIGN}


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](dict(case), int(seed))


def run(state):
    return state["pass"]()


def _prepare_layer(c, seed):
    t, gen = _Tables(c, seed), _gen(seed)
    pb, L = t.pb, t.layer(c, gen)
    out = torch.zeros_like(L["q"])
    pb.allocate_initial()
    keep, strategy = c["keep"], STRATEGY[c["strategy"]]

    def one_pass():
        # attention, masses, S += s, and the prune event that writes the next layer's table (this layer's stays)
        pb.layer(L["q"], L["k_self"], L["v_self"], L["k_store"], L["v_store"], out, keep=keep, strategy=strategy)
        return [out, pb.mass, pb.score, pb.keep_idx, pb.n_keep, pb.order, pb.next_segs, pb.next_n_seg, pb.next_new_start,
                pb.next_q_start, pb.dev_flag]

    return {"pass": one_pass}


def _prepare_stack(c, seed):
    t, gen = _Tables(c, seed), _gen(seed)
    pb = t.pb
    layers = [t.layer(c, gen) for _ in range(c["layers"])]
    outs = torch.zeros((c["layers"], *layers[0]["q"].shape), dtype=layers[0]["q"].dtype, device="cuda")
    out_of = list(outs)
    keeps, strategy = _alive(c)[1], STRATEGY[c["strategy"]]
    cand0 = torch.arange(pb.stride, dtype=torch.int32, device="cuda").repeat(pb.batch, 1)

    def one_pass():
        # a new query: every document is a candidate again
        pb.cand.copy_(cand0)
        pb.n_cand.fill_(pb.stride)
        pb.score.zero_()
        pb.n_alive = pb.stride
        pb.allocate_initial()
        for i, L in enumerate(layers):
            keep = keeps.get(i)
            pb.layer(L["q"], L["k_self"], L["v_self"], L["k_store"], L["v_store"], out_of[i], keep=keep, strategy=strategy,
                     defer=keep is None)
            if keep is not None:
                pb.advance()
        return [outs, pb.mass, pb.score, pb.segs, pb.n_seg, pb.q_start, pb.n_cand, pb.n_reuse, pb.dev_flag]

    return {"pass": one_pass}


def _prepare_decode(c, seed):
    gen, b = _gen(seed), c["batch"]
    lens = _lens(c, b, seed + 1)
    off = np.concatenate([[0], np.cumsum(lens)])
    tokens = int(off[-1])
    desc = _desc(c, tokens)
    k_cache, v_cache = (_normal(gen, _store_shape(c, tokens), c["dtype"]) for _ in range(2))
    q = _normal(gen, (b, c["hq"], c["d"]), c["dtype"])
    k1, v1 = (_normal(gen, (b, c["hkv"], c["d"]), c["dtype"]) for _ in range(2))
    # every query: its run of the cache, already at final positions, and the new token right behind it
    p_new = int(min(lens.max(), c["positions"] - 1))
    table = cf.segments_to_device(cf.segments_array(
        [s for i in range(b) for s in ((int(off[i]), int(lens[i]), 0, 0, cf.CF_SEG_PREFIX, -1),
                                       (i, 1, p_new, p_new, cf.CF_SEG_SELF, -1))]))
    n_seg = torch.full((b,), 2, dtype=torch.int32, device="cuda")
    q_off = torch.arange(b + 1, dtype=torch.int32, device="cuda")
    q_new = torch.full((b,), p_new, dtype=torch.int32, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = torch.zeros_like(q)
    max_kv = int(lens.max()) + 1
    ws_bytes = cf.cf_prefill_workspace_bytes(desc, b, 1, 2, max_kv)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")

    def one_pass():
        cf.cf_prefill_attention(desc, q, q_off, p_new, q_new, k_cache, v_cache, tokens, k1, v1, table, n_seg, 2, b, 1, max_kv,
                                out, None, None, 1, ws, ws_bytes, flag)
        return [out, flag]

    return {"pass": one_pass}


def _prepare_encode(c, seed):
    gen, n = _gen(seed), c["docs"]
    lens = _lens(c, n, seed + 1)
    off = c["prefix"] + np.concatenate([[0], np.cumsum(lens)])
    tokens = int(off[-1])
    desc = _desc(c, tokens)
    sb = pl.StoreBuilder(desc, off[:-1], lens, np.full(n, c["prefix"]), c["prefix"], tokens)
    q, k, v = (_normal(gen, (int(lens.sum()), h, c["d"]), c["dtype"]) for h in (c["hq"], c["hkv"], c["hkv"]))
    k_store, v_store = (_normal(gen, _store_shape(c, tokens), c["dtype"]) for _ in range(2))    # the prefix is encoded already
    ts, hs = pl.store_strides(tokens, c["hkv"], c["d"], c["layout"])
    out = torch.zeros_like(q)

    def one_pass():
        sb.attend(q, k, v, k_store, v_store, out)
        sb.write(k, v, k_store, v_store, ts, hs)
        return [out, k_store, v_store, sb.final_len, sb.dev_flag]

    return {"pass": one_pass}


def _prepare_assemble(c, seed):
    t, gen = _Tables(c, seed), _gen(seed)
    pb, L = t.pb, t.layer(c, gen)
    pb.allocate_initial()
    runs = c["prefix"] + t.doc_len.sum(axis=1) + c["tq"]
    off = np.concatenate([[0], np.cumsum(runs)])
    total = int(off[-1])
    final_off = torch.from_numpy(off[:-1].astype(np.int64)).cuda()
    final_len = torch.zeros(c["batch"], dtype=torch.int32, device="cuda")
    final_pos = torch.zeros(total, dtype=torch.int32, device="cuda")
    k_final, v_final = (torch.zeros((c["hkv"], total, c["d"]), dtype=TORCH[c["dtype"]], device="cuda") for _ in range(2))
    fts, fhs = pl.store_strides(total, c["hkv"], c["d"], "head")
    max_seg = int(max(t.doc_len.max(), c["prefix"], c["tq"]))

    def one_pass():
        cf.cf_assemble_cache(t.desc, L["k_store"], L["v_store"], t.n_tokens, L["k_self"], L["v_self"], pb.q_off, pb.segs, pb.n_seg,
                             pb.seg_stride, pb.batch, pb.tq, max_seg, final_off, total, fts, fhs, k_final, v_final, final_len,
                             final_pos, pb.dev_flag)
        return [k_final, v_final, final_len, final_pos, pb.dev_flag]

    return {"pass": one_pass}


def _prepare_reposition(c, seed):
    gen, n = _gen(seed), c["docs"]
    lens = _lens(c, n, seed + 1)
    off = np.concatenate([[0], np.cumsum(lens)])
    tokens = int(off[-1])
    desc = _desc(c, tokens)
    keys = _normal(gen, _store_shape(c, tokens), c["dtype"])
    moved = torch.zeros_like(keys)
    room = c["positions"] - lens
    new = (np.random.default_rng(seed + 2).random(n) * room).astype(np.int64)
    segs = cf.segments_to_device(cf.segments_array(
        [(int(off[i]), int(lens[i]), min(32, int(room[i])), int(new[i]), cf.CF_SEG_DOC, i) for i in range(n)]))
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    longest = int(lens.max())

    def one_pass():
        cf.cf_reposition_keys(desc, keys, moved, segs, n, tokens, longest, flag)
        return [moved, flag]

    return {"pass": one_pass}
