"""GPU parity of the streaming kernels (cf_reposition_keys, cf_assemble_cache) where the numbering of their work items can
go wrong: the last piece of a segment, one or two items per thread, segments past the stated longest length, more than 2^20
items in one segment, either store layout."""

import numpy as np
import pytest
import torch

from oracle import cachefocus_oracle as orc
from paper_2502_11101_amd import binding as cf
from paper_2502_11101_amd import pipeline as pl
from paper_2502_11101_amd import workloads as wl

pytestmark = pytest.mark.gpu

I32 = dict(dtype=torch.int32, device="cuda")
HALF, INTER = cf.CF_ROPE_HALF, cf.CF_ROPE_INTERLEAVED
TOL = {"f32": 2e-6, "bf16": 2.0 ** -8, "f16": 2.0 ** -10}      # one rounding of the result (fp32: of the angle and products)

# lengths, stated longest length, kv heads, head size
SHAPES = [
    ([1], 1, 1, 16),                    # one item
    ([7, 0, 13, 64], 64, 5, 48),        # three items per row, pieces that end inside a row's heads
    ([33, 150, 2], 40, 32, 128),        # a segment longer than stated
    ([200] * 19 + [101], 200, 32, 128), # many pieces
    ([2060, 3], 2060, 32, 256),         # more items than are numbered together
    ([150] * 30 + [2], 40, 32, 128),    # two items per thread in the assembly, segments longer than stated
    ([33, 150, 2], 100000, 32, 128),    # stated far too long: fewer pieces than that would take
    ([1, 2, 3] * 3000 + [500], 500, 2, 32),   # more segments than a launch has blocks for pieces: one each, in rounds
]


def _case(lens, hkv, d, dtype, layout):
    rng = np.random.default_rng(sum(lens) + d)
    n = sum(lens) + 3
    k, v = (wl.round_to_dtype(rng.standard_normal((n, hkv, d), dtype=np.float32), dtype) for _ in range(2))
    off = np.concatenate([[0], np.cumsum(lens)]) + 2
    segs = [orc.Segment(int(off[i]), l, 5, int(rng.integers(0, 2000)) if i else 1999, cf.CF_SEG_DOC, i) for i, l in enumerate(lens)]
    ts, hs = pl.store_strides(n, hkv, d, layout)
    return n, k, v, segs, (ts, hs)


def _tokens_first(t, layout):
    return (t if layout == "token" else t.transpose(0, 1)).float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("layout", ["token", "head"])
@pytest.mark.parametrize("dtype,pairing", [("bf16", HALF), ("f16", INTER), ("f32", HALF), ("f32", INTER)])
@pytest.mark.parametrize("lens,longest,hkv,d", SHAPES)
def test_moves(lens, longest, hkv, d, dtype, pairing, layout):
    print(f"moves lens={lens[:4]} hkv={hkv} d={d} {dtype} pairing={pairing} {layout}", flush=True)
    n, k, v, segs, (ts, hs) = _case(lens, hkv, d, dtype, layout)
    desc = cf.make_desc(hkv, hkv, d, dtype, 1.0e4, 8192, pairing, store_token_stride=ts, store_head_stride=hs)
    k_dev, v_dev = (pl.store_to_device(x, dtype, layout) for x in (k, v))
    table, flag = cf.segments_to_device(cf.segments_array(segs)), torch.zeros(1, **I32)
    ref = orc.reposition_keys(k, segs, 1.0e4, "half" if pairing == HALF else "interleaved")
    bound = TOL[dtype] * max(1.0, np.abs(ref).max())

    moved = k_dev.clone()
    cf.cf_reposition_keys(desc, k_dev, moved, table, len(segs), n, longest, flag)
    got = _tokens_first(moved, layout)
    assert np.max(np.abs(got - ref)) <= bound
    assert np.array_equal(got[:2], k[:2]) and np.array_equal(got[-1], k[-1])          # listed by no segment

    total = sum(lens)
    k_out, v_out = (torch.full((n, hkv, d) if layout == "token" else (hkv, n, d), 3.0, dtype=k_dev.dtype, device="cuda") for _ in range(2))
    final_len, pos = torch.zeros(1, **I32), torch.full((n,), -1, **I32)
    cf.cf_assemble_cache(desc, k_dev, v_dev, n, None, None, torch.zeros(2, **I32), table, torch.full((1,), len(segs), **I32),
                         len(segs), 1, 1, longest, torch.ones(1, dtype=torch.int64, device="cuda"), n, ts, hs, k_out, v_out,
                         final_len, pos, flag)
    got_k, got_v = _tokens_first(k_out, layout), _tokens_first(v_out, layout)
    rows = slice(1, 1 + total)
    src = slice(2, 2 + total)
    assert final_len.item() == total and flag.item() == 0
    assert np.max(np.abs(got_k[rows] - ref[src]), initial=0.0) <= bound
    assert np.array_equal(got_v[rows], v[src].astype(np.float64))
    assert np.all(got_k[0] == 3.0) and np.all(got_v[0] == 3.0) and np.all(got_k[1 + total:] == 3.0) and np.all(got_v[1 + total:] == 3.0)
    want = np.concatenate([np.arange(s.new_start, s.new_start + s.len) for s in segs])
    assert pos[rows].cpu().numpy().tolist() == want.tolist()


def _median_us(call):
    times = []
    for _ in range(9):
        e0, e1 = torch.cuda.Event(True), torch.cuda.Event(True)
        e0.record()
        for _ in range(20):
            call()
        e1.record()
        torch.cuda.synchronize()
        times.append(e0.elapsed_time(e1) * 50)
    return sorted(times)[4]


def test_a_long_table_is_not_added_up_by_every_piece():
    """2000 documents of 20 tokens: the blocks of the assembly each add up the table, so they are few; the time stays within a small
    multiple of the re-positioning's (half the bytes, no table): 4 times, over 9 with as many blocks as pieces."""
    n_seg, length, hkv, d = 2000, 20, 8, 128
    n = n_seg * length
    ts, hs = pl.store_strides(n, hkv, d, "head")
    desc = cf.make_desc(hkv, hkv, d, "bf16", 1.0e4, 1 << 20, HALF, store_token_stride=ts, store_head_stride=hs)
    table = cf.segments_to_device(cf.segments_array([(i * length, length, 5, 9 * i, cf.CF_SEG_DOC, i) for i in range(n_seg)]))
    k = torch.randn(n * hkv * d, device="cuda").to(torch.bfloat16)
    k_out, v_out, flag = torch.empty_like(k), torch.empty_like(k), torch.zeros(1, **I32)
    q_off, count, final_off, final_len = torch.zeros(2, **I32), torch.full((1,), n_seg, **I32), torch.zeros(1, dtype=torch.int64, device="cuda"), torch.zeros(1, **I32)
    moved = _median_us(lambda: cf.cf_reposition_keys(desc, k, k_out, table, n_seg, n, length, flag))
    assembled = _median_us(lambda: cf.cf_assemble_cache(desc, k, k, n, None, None, q_off, table, count, n_seg, 1, 1, length, final_off, n, ts, hs,
                                                        k_out, v_out, final_len, None, flag))
    print(f"long table: re-positioning {moved:.1f} us, assembly {assembled:.1f} us", flush=True)
    assert flag.item() == 0 and final_len.item() == n
    assert torch.equal(v_out, k)
    assert assembled <= 7 * moved


def test_a_loose_stated_length_costs_little():
    """The stated longest length only sizes the launch: a bound 200 times too large may not cost a multiple of the call."""
    n_seg, length, hkv, d = 30, 160, 32, 128
    n = n_seg * length
    ts, hs = pl.store_strides(n, hkv, d, "head")
    desc = cf.make_desc(hkv, hkv, d, "bf16", 1.0e4, 8192, HALF, store_token_stride=ts, store_head_stride=hs)
    table = cf.segments_to_device(cf.segments_array([(i * length, length, 5, 9 * i, cf.CF_SEG_DOC, i) for i in range(n_seg)]))
    k = torch.randn(n * hkv * d, device="cuda").to(torch.bfloat16)
    k_out, v_out, flag = torch.empty_like(k), torch.empty_like(k), torch.zeros(1, **I32)
    q_off, count, final_off, final_len = torch.zeros(2, **I32), torch.full((1,), n_seg, **I32), torch.zeros(1, dtype=torch.int64, device="cuda"), torch.zeros(1, **I32)

    def moved(longest):
        cf.cf_reposition_keys(desc, k, k_out, table, n_seg, n, longest, flag)

    def assembled(longest):
        cf.cf_assemble_cache(desc, k, k, n, None, None, q_off, table, count, n_seg, 1, 1, longest, final_off, n, ts, hs, k_out, v_out, final_len, None, flag)

    for call in (moved, assembled):
        fits, loose = (_median_us(lambda: call(longest)) for longest in (length, 200 * length))
        print(f"{call.__name__}: {fits:.1f} us, stated 200 times longer {loose:.1f} us", flush=True)
        assert loose <= 3 * fits             # (without a limit on the launch: over 20 times)
    assert flag.item() == 0
