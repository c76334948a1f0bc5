"""Calls with a workspace that was sized for other bounds: larger ones (a decode loop's longest cache) and, where the bytes allow it,
smaller ones, whose calls go without the runs of tiles and row groups that do not fit."""

import pytest

from paper_2502_11101_amd import binding as cf
from tests import gpu_harness as G
from tests import plan_probe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,batch", [(32, 32, 1), (28, 4, 8)])
@pytest.mark.parametrize("n", [300, 831, 1000, 1215])
def test_one_workspace_for_a_growing_cache(hq, hkv, batch, n):
    print(f"workspace for 4096 tokens, {batch} x {n}, {hq}/{hkv}", flush=True)
    d = cf.make_desc(hq, hkv, 128, "bf16", 1.0e4, 8192, cf.CF_ROPE_HALF)
    G.check_tables(hq, hkv, 1, [[(0, n, 0, 0)]] * batch, n, "bf16", n, seed=n, given=cf.cf_prefill_workspace_bytes(d, batch, 1, 2, 4096))


# a decode step of eight runs per split; four row groups of two blocks; two groups of wavefronts
@pytest.mark.parametrize("hq,hkv,batch,tq,lens", [(32, 32, 1, 1, [1000]), (28, 4, 1, 20, [3000]), (12, 2, 64, 32, [1000, 90])])
def test_the_least_workspace(hq, hkv, batch, tq, lens):
    print(f"least workspace {hq}/{hkv} {batch} x {tq}", flush=True)
    args = (hq, hkv, batch, tq, len(lens) + 1, sum(lens) + tq)
    least, best = plan_probe.plan(*args, given=0), plan_probe.plan(*args)
    assert least.total < best.total
    table = [(0, lens[0], 16, 900)] + [(lens[0], n, 16, 16) for n in lens[1:]]
    G.check_tables(hq, hkv, tq, [table] * batch, sum(lens), "bf16", 0, seed=tq, check=sorted({0, batch - 1}), given=least.total)
