"""Launch plans of the 16-bit attention path, as far as the host sees them."""

import pytest

from paper_2502_11101_amd import binding as cf
from tests import attn_cases, plan_probe


def test_static_calls_of_many_rows_stay_accepted():
    """Calls of many stacked rows whose plan of at most twelve row blocks a group, one slot per entry and split, fits the static entry
    point's buffer: the plan in use, which may have a second group of wavefronts (one more slot per split), fits it as well."""
    up = lambda x: -(-x // 256) * 256
    limit, near = cf.CF_STATIC_SCRATCH_BYTES, 0
    for hq, hkv in ((28, 4), (12, 2), (32, 8), (32, 32)):
        d = cf.make_desc(hq, hkv, 128, "bf16", 1.0e4, 32768, cf.CF_ROPE_HALF)
        for batch in (*range(1, 24), 32, 48, 64, 100, 128, 200):
            for tq in (24, 48, 64, 100, 180):
                for stride in (*range(3, 66, 9), *range(70, 257, 6)):
                    for max_kv in (500, 8000):
                        blocks = -(-hq // hkv * tq // 16)
                        if blocks <= 4:
                            continue
                        units = batch * hkv * -(-blocks // 12)
                        splits = max(1, min(256 // units, (max_kv // 32 + stride) // 2, 32))
                        slots = stride + splits
                        total = up(units * splits * 1536) + (up(units * splits * 49152) if splits > 1 else 0) + up(units * slots * 1536) + \
                            16 * up(units * 3 * slots * 4)
                        if total <= limit:
                            need = cf.cf_prefill_workspace_bytes(d, batch, tq, stride, max_kv)
                            assert need <= limit, (hq, hkv, batch, tq, stride, max_kv)
                            near += total > limit - (1 << 20)
    assert near > 10


def test_row_groups_stay_within_the_grid():
    """A call whose (kv heads x row groups) the grid holds only with the larger row groups gets those: 28 row blocks of 20000 kv
    heads are three groups of three blocks per wavefront (60000), where groups of two would be four (80000)."""
    up = lambda x: -(-x // 256) * 256
    d = cf.make_desc(20000, 20000, 128, "bf16", 1.0e4, 32768, cf.CF_ROPE_HALF)
    units, slots = 20000 * 3, 3 + 1
    want = up(units * 192 * 8) + up(units * slots * 192 * 8) + 16 * up(units * 3 * slots * 4)
    assert cf.cf_prefill_workspace_bytes(d, 1, 448, 3, 4000) == want


def test_the_grid_holds_what_the_header_says():
    """n_kv_heads x row groups of up to 192 rows <= 65535: one row block of 65535 heads, and 193 rows (two groups) of 32767; not one more of either."""
    for hkv, tq, fits in ((65535, 4, 1), (65536, 4, 0), (32767, 193, 1), (32768, 193, 0), (21845, 385, 1)):
        assert plan_probe.plan(hkv, hkv, 1, tq, 3, 4000).grid_ok == fits, (hkv, tq)


def test_static_calls_of_one_row_block_stay_accepted():
    """As above for one 16-row block: a plan of two runs of tiles per workgroup that fits the static entry point's buffer; the plan in use
    may have eight (six more slots per split)."""
    up = lambda x: -(-x // 256) * 256
    limit, near = cf.CF_STATIC_SCRATCH_BYTES, 0
    for hkv in (1, 2, 4, 32):
        d = cf.make_desc(2 * hkv, hkv, 128, "bf16", 1.0e4, 32768, cf.CF_ROPE_HALF)
        for batch in (*range(1, 24), 32, 40, 64, 100, 128, 200, 500, 1000, 2000):
            for stride in (*range(1, 66, 9), *range(70, 257, 6)):
                for max_kv in (100, 500, 2000, 8000):
                    units, tiles = batch * hkv, max_kv // 32 + stride
                    splits = 2 if 128 < units < 192 and tiles > 128 else max(1, min(256 // units, max(tiles // 4, 1), 32))
                    slots = stride + 2 * splits
                    total = up(units * splits * 512) + (up(units * splits * 16384) if splits > 1 else 0) + up(units * slots * 512) + \
                        16 * up(units * slots * 4)
                    if total <= limit:
                        need = cf.cf_prefill_workspace_bytes(d, batch, 8, stride, max_kv)
                        assert need <= limit, (hkv, batch, stride, max_kv)
                        near += total > limit - (1 << 20)
    assert near > 10


@pytest.mark.parametrize("hq,hkv", [(32, 32), (28, 4), (12, 2), (8, 1), (32, 8)])
def test_a_workspace_for_the_longest_lists_serves_all_shorter_ones(hq, hkv):
    """The bytes reported never shrink as max_kv_tokens or seg_stride grows, and the plan of a call needs no more than is reported for
    its own arguments: what was allocated for a decode loop's longest cache serves every step on the way."""
    d = cf.make_desc(hq, hkv, 128, "bf16", 1.0e4, 32768, cf.CF_ROPE_HALF)
    tokens = [*range(0, 1600, 32), 2000, 3000, 4096, 8000, 12000, 30000]
    for batch in (1, 2, 3, 8, 24, 32, 33, 48, 64, 200):
        for tq in (1, 4, 20, 48, 64, 130):
            shorter = [0] * len(tokens)                  # the bytes of the table before, per number of tokens
            for stride in (1, 2, 3, 4, 12, 52, 65, 200):
                last = 0
                for i, kv in enumerate(tokens):
                    need = cf.cf_prefill_workspace_bytes(d, batch, tq, stride, kv)
                    assert need >= last and need >= shorter[i], (batch, tq, stride, kv)
                    last = shorter[i] = need
                    assert plan_probe.plan(hq, hkv, batch, tq, stride, kv, need).total <= need, (batch, tq, stride, kv)


def test_a_decode_loop_allocates_once():
    """One workspace, sized for 4096 tokens: no shorter cache is refused for it.  (The call ends at the next check, of the pointer.)"""
    fake = 0x1000                                        # never dereferenced
    for hq, hkv, batch in ((32, 32, 1), (28, 4, 8)):
        d = cf.make_desc(hq, hkv, 128, "bf16", 1.0e4, 8192, cf.CF_ROPE_HALF)
        have = cf.cf_prefill_workspace_bytes(d, batch, 1, 2, 4096)
        for kv in range(1, 4097, 31):
            with pytest.raises(cf.CacheFocusError) as e:
                cf.cf_prefill_attention(d, fake, fake, 0, fake, fake, fake, 5000, fake, fake, fake, fake, 2, batch, 1, kv, fake, None, None, 1,
                                        0x10010, have, None, stream=0)
            assert "aligned" in e.value.message, (kv, e.value.message)


def test_the_attention_tests_reach_every_variant():
    """The calls of attn_cases get the plans written beside them; those of many rows take every combination of blocks per wavefront, groups of
    wavefronts, table form, and one split or several, and the CAUSAL variant with either number of blocks."""
    for c in attn_cases.WIDE:
        p = plan_probe.plan(c.group * c.hkv, c.hkv, c.batch, c.tq, c.entries, c.tokens)
        assert (p.wide, p.nrb, p.groups, p.n_rg, p.nsplit) == (1 + c.causal, c.nrb, c.groups, c.n_rg, c.nsplit), c
    assert {(c.nrb, c.groups, c.entries <= 64, c.nsplit == 1) for c in attn_cases.WIDE if not c.causal} == \
        {(n, g, reg, one) for n in (2, 3) for g in (1, 2) for reg in (True, False) for one in (True, False)}
    assert {c.nrb for c in attn_cases.WIDE if c.causal} == {2, 3}
    for c in attn_cases.SOLO:
        p = plan_probe.plan(c.hq, c.hkv, c.batch, c.tq, 2, c.tokens)
        assert (p.groups, p.nsplit, -(-(c.tokens // 32 + 2) // (8 * p.nsplit))) == (8, c.nsplit, c.tiles), c


def test_a_split_pays_for_its_merge():
    """Documents encoded over a 32-token prefix: eight row groups in one split, not five in two that save three tiles; one group of wavefronts
    where a split has ten tiles of three blocks each, two from thirteen on, and from ten on with five blocks in all.  Long lists are split as before."""
    shape = lambda *a: plan_probe.plan(*a)[1:5]          # blocks per wavefront, groups, row groups, splits
    assert shape(12, 2, 12, 160, 2, 192) == (2, 1, 8, 1)
    assert shape(12, 2, 16, 228, 2, 260) == (3, 1, 8, 1)
    assert shape(12, 2, 6, 340, 2, 372) == (2, 2, 16, 1)
    assert shape(32, 16, 8, 40, 5, 492) == (2, 2, 1, 2)
    assert shape(28, 4, 1, 64, 52, 7446) == (2, 2, 4, 16)


def test_decode_calls_of_many_rounds_keep_the_tile_kernel():
    """attn_solo_kernel (eight runs of tiles per workgroup) up to 1024 units."""
    for tokens in (300, 600, 2000):
        assert plan_probe.plan(32, 32, 32, 1, 2, tokens).groups == 8
        assert plan_probe.plan(32, 32, 33, 1, 2, tokens).groups == 2


# dtype, pairs, query heads, kv heads, head_dim, rows, table entries, tokens; queries of the workspace and of the call
@pytest.mark.parametrize("case", [("f32", "half", 12, 2, 128, 100, 7, 536, 2, 1), ("bf16", "interleaved", 32, 8, 128, 20, 32, 1500, 2, 1),
                                  ("f32", "half", 12, 2, 64, 8, 2, 536, 16, 8), ("bf16", "half", 28, 4, 96, 8, 2, 800, 8, 6)])
def test_a_workspace_for_more_queries_serves_fewer_on_the_fp32_precision_path(case):
    """Where a call runs in eight splits though more would fill the device, the bytes of those are reported: a smaller batch, which may have them, is
    served by the workspace of the larger one.  (The calls end at the next check, of the pointer.)"""
    dtype, pairs, hq, hkv, dim, tq, stride, kv, many, few = case
    fake = 0x1000                                        # never dereferenced
    d = cf.make_desc(hq, hkv, dim, dtype, 1.0e4, 8192, cf.CF_ROPE_INTERLEAVED if pairs == "interleaved" else cf.CF_ROPE_HALF)
    have = cf.cf_prefill_workspace_bytes(d, many, tq, stride, kv)
    for batch in (few, many):
        with pytest.raises(cf.CacheFocusError) as e:
            cf.cf_prefill_attention(d, fake, fake, 0, fake, fake, fake, 9000, fake, fake, fake, fake, stride, batch, tq, kv, fake, None, None, 1,
                                    0x10010, have, None, stream=0)
        assert "aligned" in e.value.message, (batch, e.value.message)
