"""CPU-only checks of the split rules of the decode steps (tests/decode_rules.py compiles them from the library's own source)."""
import ctypes as C

import numpy as np
import pytest

from paper_2602_07529_amd import binding as B
from tests import decode_rules


def test_the_rules_are_those_of_the_library():
    rng = np.random.default_rng(8)
    for _ in range(200):
        groups, hkv, g, size = (int(rng.integers(1, x)) for x in (17, 9, 9, 33))
        d, shared, own = int(rng.choice([64, 128])), int(2 ** rng.uniform(0, 11)), int(2 ** rng.uniform(0, 7))
        desc = B.dag_decode_desc_t(groups, groups * size, 16, shared, own, size, *([0x1000] * 8))
        assert decode_rules.decode(desc, hkv * g, hkv, d).bytes == B.lib().dag_decode_workspace_bytes(C.byref(desc), hkv * g, hkv, d)
        seg = B.dag_decode_seg_desc_t(groups * size, groups + groups * size, 16, max(shared, own), size, 2 * groups * size, *([0x1000] * 8))
        assert decode_rules.segments(seg, hkv * g, hkv, d).bytes == B.lib().dag_decode_segments_workspace_bytes(C.byref(seg), hkv * g, hkv, d)


# Sibling groups of more than 32 rows: shared slices x pages, own slices x pages; False: the slices that the workspace is sized for.
@pytest.mark.parametrize("groups,nb,shared,own,hq,hkv,d,want,lengthened", [
    (8, 17, 1488, 4, 8, 2, 64, (16, 96, 1, 64), True),       # a workgroup for every compute unit, not half of them in slices of 128
    (7, 21, 706, 29, 20, 4, 64, (9, 80, 1, 64), True),
    (3, 20, 395, 7, 32, 8, 128, (5, 80, 1, 64), True),       # 120 workgroups
    (1, 22, 817, 13, 8, 4, 128, (26, 32, 3, 6), True),       # 104: 33 partials would be two rounds of the merge
    (1, 22, 817, 10, 8, 4, 128, (30, 28, 2, 6), True),       # 120: 32 are one
    (2, 20, 976, 57, 16, 2, 128, (28, 36, 4, 16), True),     # 112: 35 would be two
    (1, 31, 1245, 8, 8, 2, 64, (52, 24, 2, 4), True),        # 65 at dimension 64
    (2, 23, 335, 9, 5, 1, 64, (42, 8, 2, 6), False),         # few workgroups with little each: slices of eight pages
    (2, 21, 1091, 9, 3, 1, 128, (55, 20, 2, 6), True),       # 55 workgroups to a group
    (12, 14, 241, 75, 5, 1, 128, (7, 36, 2, 38), True),      # 84 workgroups beside 168 with own pages
    (4, 26, 144, 87, 20, 4, 128, (3, 48, 2, 44), True),      # 48 beside 208
    (8, 10, 79, 93, 8, 2, 128, (5, 16, 2, 48), True) ,        # own pages are most of it
    (12, 19, 696, 28, 8, 2, 128, (10, 72, 1, 64), True),     # slices of 128 pages would be 144 workgroups
    (10, 10, 128, 17, 32, 8, 128, (1, 128, 1, 64), True),    # 80 workgroups: not too many
    (1, 29, 59, 37, 48, 8, 128, (8, 8, 3, 16), False),       # 64 and 174 workgroups: all at once
    (2, 32, 2048, 40, 40, 8, 128, (16, 128, 1, 64), False),
])
def test_slices_of_wide_groups(groups, nb, shared, own, hq, hkv, d, want, lengthened):
    p = decode_rules.step(groups, nb, shared, own, hq, hkv, d)
    assert (p.splits_a, p.chunk_a, p.splits_b, p.chunk_b) == want
    assert p.route == "wide" and (p.settle < 1024) == lengthened and p.chunk_a % 4 == 0


def test_wide_groups_without_a_shared_context_are_enough_single_waves():
    for groups, nb, own, hq, hkv in ((1, 30, 500, 8, 1), (2, 20, 300, 16, 2), (1, 12, 4000, 24, 4)):
        p = decode_rules.step(groups, nb, 0, own, hq, hkv, 128)
        assert p.route == "items" and groups * nb * hkv * p.splits_b >= 512


def test_rules_never_make_more_partials_than_the_workspace_holds():
    rng = np.random.default_rng(9)
    for _ in range(4000):
        groups, hkv, g, size = (int(rng.integers(1, x)) for x in (40, 9, 33, 70))
        d, shared, own = int(rng.choice([64, 128])), int(2 ** rng.uniform(0, 13)) - 1, int(2 ** rng.uniform(0, 9)) - 1
        p = decode_rules.step(groups, size, shared, own, hkv * g, hkv, d)
        assert p.splits_a * p.chunk_a >= shared and p.splits_b * p.chunk_b >= own and p.chunk_a % 2 == 0 and p.chunk_b % 2 == 0
        assert not p.wide or p.chunk_a <= 128
        rows = groups * hkv * p.rb_max * p.splits_a * 32 + groups * size * hkv * p.splits_b * g
        assert rows * (d + 2) * 4 + 256 <= p.bytes


# Single waves: slices get longer where the merge goes round once less (32 partials at head dimension 128, 64 at 64, 16 in many rows) or
# where the last one would be an eighth of 16 pages or more, and not where a step is one chain of a few blocks.
@pytest.mark.parametrize("groups,nb,shared,own,hq,hkv,d,want", [
    (1, 4, 94, 16, 32, 8, 128, (12, 8, 4, 4)),       # 16 partials either way
    (1, 1, 211, 5, 2, 1, 128, (27, 8, 2, 4)),
    (2, 5, 29, 41, 5, 1, 128, (4, 8, 11, 4)),
    (1, 1, 509, 43, 8, 1, 128, (51, 10, 8, 6)),      # 75 -> 59
    (1, 1, 509, 43, 8, 1, 64, (51, 10, 8, 6)),       # 75 -> 59: two rounds -> one
    (1, 1, 747, 49, 2, 2, 64, (94, 8, 13, 4)),       # 107 -> 84: two either way
    (16, 32, 257, 4, 16, 16, 128, (2, 130, 1, 64)),   # a last page of 128: joined
    (16, 32, 275, 4, 16, 16, 128, (3, 128, 1, 64)),   # 19 pages are not
    (3, 3, 17, 0, 4, 1, 128, (3, 8, 0, 4)),
])
def test_slices_of_single_waves(groups, nb, shared, own, hq, hkv, d, want):
    p = decode_rules.step(groups, nb, shared, own, hq, hkv, d)
    assert not p.wide and (p.splits_a, p.chunk_a, p.splits_b, p.chunk_b) == want
    assert p.th == 3 or p.route == "whole"   # at 1 frontiers of many rows took 2 to 6 % longer


# A (branch, KV head) to a workgroup: where the shared pages are few enough to be read by every branch.
@pytest.mark.parametrize("groups,nb,shared,own,hq,hkv,d,whole", [
    (1, 4, 32, 20, 32, 8, 128, True), (1, 4, 33, 20, 32, 8, 128, False),
    (1, 4, 41, 5, 32, 8, 128, True), (1, 4, 42, 5, 32, 8, 128, False),
    (1, 4, 40, 56, 32, 8, 64, True), (1, 4, 40, 57, 32, 8, 64, False), (1, 4, 57, 2, 32, 8, 64, False),
    (1, 9, 62, 2, 32, 8, 128, True), (1, 9, 62, 3, 32, 8, 128, False),            # two row blocks
    (2, 9, 76, 20, 32, 8, 64, True), (2, 9, 77, 19, 32, 8, 64, False),
    (16, 8, 35, 4, 4, 1, 128, False), (16, 1, 35, 4, 4, 1, 128, True),            # siblings on eight dies; no siblings
    (2, 8, 35, 4, 32, 8, 128, True), (2, 8, 35, 4, 20, 5, 128, False), (2, 8, 35, 4, 16, 4, 128, True),
    (4, 8, 7, 7, 9, 1, 128, False), (4, 8, 7, 7, 8, 1, 128, True),                # nine rows a branch
    (2, 16, 7, 7, 8, 8, 128, True), (1, 33, 7, 7, 8, 8, 128, False),              # 256 workgroups
])
def test_short_contexts_that_a_workgroup_takes_whole(groups, nb, shared, own, hq, hkv, d, whole):
    assert (decode_rules.step(groups, nb, shared, own, hq, hkv, d).route == "whole") == whole
