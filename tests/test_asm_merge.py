"""Static check of the segment merge: a partial output is added to the sum in one rounding (fused multiply-add), for
each of the eight partials that are in flight together."""
import os

import pytest

from tests.test_asm_lds_reads import HIPCC, _assembly, _kernels


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_segment_merge_adds_partials_with_one_rounding(tmp_path):
    seen = 0
    for name, lines in _kernels(_assembly("decode", tmp_path), "k_decode_seg_merge"):
        per_lane = 2 if "ILi128E" in name else 1
        fused = sum(1 for l in lines if l.strip().startswith(("v_fma_f32", "v_fmac_f32")))
        # (the index and output divisions and the running sum of the weights take eight of their own)
        assert fused >= 7 * per_lane + 8, "%s: %d" % (name, fused)
        seen += 1
    assert seen == 2
