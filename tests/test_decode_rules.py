"""CPU-only checks of the split rules of the decode steps (tests/decode_rules.py compiles them from the library's own source)."""
import ctypes as C

import numpy as np

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
