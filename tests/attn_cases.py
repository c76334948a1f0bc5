"""Calls that reach every variant of the 16-bit attention kernels for many stacked rows and for one row block, each with what the launch
plan makes of it.  The GPU tests run them; tests/test_plan_host.py holds the plan to what is written here, so that a change of
the plan cannot leave a variant without a test."""

from collections import namedtuple

# rows: stacked rows of a kv head (group x tq); entries and tokens: the longest table of the batch, own block included
# plan: 16-row blocks per wavefront (nrb), groups of wavefronts, row groups, splits, and whether the CAUSAL variant runs
Wide = namedtuple("Wide", "group hkv batch tq entries tokens nrb groups n_rg nsplit causal", defaults=(0,))
WIDE = [
    # table in registers
    Wide(4, 2, 3, 32, 3, 200, 2, 1, 1, 2),           # 128 rows: eight blocks
    Wide(4, 3, 43, 32, 3, 200, 2, 1, 1, 1),          # 128, one split
    Wide(1, 3, 9, 193, 3, 1700, 2, 2, 2, 4),
    Wide(7, 2, 22, 55, 3, 1200, 2, 2, 4, 1),
    Wide(3, 3, 22, 43, 3, 900, 3, 1, 1, 3),          # 129: nine blocks, the last with one row
    Wide(6, 3, 43, 32, 3, 200, 3, 1, 1, 1),          # 192: all twelve blocks
    Wide(6, 3, 15, 32, 3, 2300, 3, 2, 1, 5),
    Wide(3, 3, 43, 43, 3, 1200, 3, 2, 1, 1),
    # CAUSAL: several row groups, or an own block of half the list
    Wide(7, 2, 22, 55, 3, 200, 2, 1, 4, 1, 1),       # 385
    Wide(2, 3, 43, 95, 3, 190, 3, 1, 1, 1, 1),       # 190
    # table in LDS
    Wide(1, 2, 1, 193, 66, 900, 2, 1, 2, 23),        # 193
    Wide(7, 2, 43, 55, 66, 900, 2, 1, 4, 1),
    Wide(7, 1, 9, 55, 66, 900, 2, 2, 4, 7),
    Wide(7, 2, 22, 55, 80, 900, 2, 2, 4, 1),
    Wide(3, 1, 22, 43, 66, 900, 3, 1, 1, 11),
    Wide(6, 3, 90, 32, 66, 900, 3, 1, 1, 1),
    Wide(6, 1, 47, 32, 66, 900, 3, 2, 1, 5),
    Wide(6, 3, 43, 32, 66, 900, 3, 2, 1, 1),
]

# one row block over at most two table entries; tiles: the most that one of a workgroup's eight wavefronts has
Solo = namedtuple("Solo", "hq hkv batch tq tokens nsplit tiles")
SOLO = [
    Solo(4, 2, 129, 1, 3300, 1, 14),
    Solo(14, 2, 70, 2, 4500, 2, 9),
    Solo(28, 4, 32, 1, 4900, 2, 10),                 # a batch of unequal conversations
    Solo(16, 1, 100, 1, 900, 1, 4),
    Solo(8, 8, 4, 4, 1000, 8, 1),
]


def id_of(c):
    return "-".join(f"{k}{v}" for k, v in c._asdict().items())
