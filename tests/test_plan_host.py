"""Launch plans of the 16-bit attention path, as far as the host sees them."""

from paper_2502_11101_amd import binding as cf


def test_two_groups_refuse_no_static_call():
    """Plans of the workspace sizes around the static entry point's buffer: a second group of wavefronts never takes one past it
    that a single group keeps within."""
    limit, seen = cf.CF_STATIC_SCRATCH_BYTES, 0
    for hq, hkv in ((28, 4), (12, 2), (32, 8)):
        d = cf.make_desc(hq, hkv, 128, "bf16", 1.0e4, 32768, cf.CF_ROPE_HALF)
        for batch in range(1, 40):
            for tq in (24, 48, 64):
                for stride in range(20, 257, 4):
                    need = cf.cf_prefill_workspace_bytes(d, batch, tq, stride, 8000)
                    group = hq // hkv
                    blocks = -(-group * tq // 16)
                    if blocks <= 4 or need <= limit:
                        continue
                    rg = -(-blocks // 12)
                    units = batch * hkv * rg
                    rows = 64 * -(-(-(-blocks // rg)) // 4)
                    splits = max(1, min(256 // units if units <= 256 else 1, 32))
                    # one group: (max, sum) pairs and partial rows, slot statistics, sixteen parts of slot masses
                    up = lambda x: -(-x // 256) * 256
                    slots = stride + splits
                    one = up(units * splits * rows * 8) + (up(units * splits * rows * 256) if splits > 1 else 0) + \
                        up(units * slots * rows * 8) + 16 * up(units * rows // 64 * slots * 4)
                    assert one > limit, (hq, hkv, batch, tq, stride)
                    seen += need < limit + (2 << 20)
    assert seen > 10
