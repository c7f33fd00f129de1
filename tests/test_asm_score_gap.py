"""Static check of the generated code of k_nodes_dkv2 (no GPU needed).

The score products of the dK / dV kernel are inline assembly, and the compiler keeps no distance between them and the vector
instructions that read their results (at most 19 wait states behind a 16-pass MFMA): the order of the source does.  Every
instruction is one state at least, `s_nop n` is n + 1.
"""
import os
import re

import pytest

from tests.test_asm_lds_reads import HIPCC, _assembly, _cfg, _kernels, _regs

STATES = 19


def _too_close(insts, carried):
    """Instructions that read or write the result of a vector-register MFMA in front of its time; `carried`: states since the write of a
    register, from the block in front.  Another MFMA that adds to the same registers is not one of them."""
    age, bad = dict(carried), []
    for l in insts:
        op, args = l.split()[0], l[len(l.split()[0]):]
        if op.startswith("v_mfma"):
            parts = re.findall(r"[va]\[\d+:\d+\]|0", args)
            if any(age.get(r, 99) < STATES for p in parts[1:3] for r in _regs(p)):
                bad.append(l)
            if any(age.get(r, 99) < STATES for r in _regs(parts[0])) and _regs(parts[0]) != _regs(parts[3]):
                bad.append(l)
        elif any(age.get(r, 99) < STATES for r in _regs(args)):
            bad.append(l)
        step = int(args, 0) + 1 if op == "s_nop" else 1
        age = {r: n + step for r, n in age.items() if n + step < STATES}
        if op.startswith("v_mfma"):
            for r in _regs(parts[0]):
                age[r] = 0
    return age, bad


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_scores_are_read_late_enough(tmp_path):
    seen = 0
    for name, lines in _kernels(_assembly("prefill_bwd", tmp_path), "k_nodes_dkv2"):
        blocks = _cfg(lines)
        entry = [{} for _ in blocks]
        for _ in range(4):  # (19 states reach over a few short blocks at most)
            for i, b in enumerate(blocks):
                age, bad = _too_close(b["insts"], entry[i])
                assert not bad, "%s: %s" % (name, bad[:3])
                for s in b["succ"]:
                    for r, n in age.items():
                        entry[s][r] = min(n, entry[s].get(r, 99))
        seen += 1
    assert seen == 1


def test_the_checker_finds_planted_mistakes():
    chain = ["v_mfma_f32_32x32x16_bf16 v[0:15], v[40:43], v[50:53], 0", "s_nop 0", "v_mfma_f32_32x32x16_bf16 v[0:15], v[44:47], v[54:57], v[0:15]"]
    use = "v_fma_f32 v60, v7, v61, v62"
    assert not _too_close(chain + ["s_nop 15", "s_nop 2", use], {})[1]
    assert _too_close(chain + ["s_nop 15", "s_nop 1", use], {})[1] == [use]
    assert _too_close(chain + [use], {})[1] == [use]
    assert _too_close([use], _too_close(chain, {})[0])[1] == [use]  # over the end of a block
    other = "v_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[50:53], a[0:15]"
    assert _too_close(chain + [other], {})[1] == [other]
