"""Sibling groups of more than 32 rows of a KV head: single-wave items where little is to be read, longer slices of the shared pages
elsewhere; and the workspace, whose size follows the shorter slices whatever the launch takes."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import dag_oracle as orc
from paper_2602_07529_amd import binding as B
from workloads import dags
from tests import decode_rules
from tests.gpu_util import DEV, check_close


def _ceil(a, b):
    return -(-a // b)


def test_workspace_sizes_follow_the_shorter_slices():
    rng = np.random.default_rng(7)
    for _ in range(400):
        groups, hkv, g, size = (int(rng.integers(1, x)) for x in (17, 9, 9, 33))
        d, shared, own = int(rng.choice([64, 128])), int(2 ** rng.uniform(0, 11)), int(2 ** rng.uniform(0, 7))
        live = groups * size
        blocks = _ceil(size * g, 32)
        wide = 2 <= blocks <= 8
        a, b = 128, 64
        while a > 8 and groups * hkv * (1 if wide else blocks) * _ceil(shared, a) < (256 if wide else 512):
            a //= 2
        while b > 4 and live * hkv * _ceil(own, b) < (512 if wide else 1024):
            b //= 2
        rows_a = groups * hkv * blocks * _ceil(shared, a) * 32
        rows_b = live * hkv * _ceil(own, b) * g
        want = sum(_ceil(x, 256) * 256 for x in (rows_a * d * 4, rows_a * 8, rows_b * d * 4, rows_b * 8)) + 256
        desc = B.dag_decode_desc_t(groups, live, 16, shared, own, size, *([0x1000] * 8))
        assert B.lib().dag_decode_workspace_bytes(C.byref(desc), hkv * g, hkv, d) == want


# groups, branches, heads per KV head, KV heads, shared tokens, longest own context; at dimensions 64 and 128 the route or, of
# k_decode_wide, the shared slices and their pages.  The error bound is that of every decode test.
@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("groups,nb,group,hkv,shared,own,want", [
    (2, 9, 4, 1, 33, 3, ("whole", "whole")),         # two row blocks, the second with four rows
    (1, 13, 5, 2, 1, 40, ("whole", "whole")),        # three; one shared token
    (2, 9, 5, 1, 1300, 3, ("items", "items")),       # two row blocks in single waves, the second with 13 rows
    (1, 13, 10, 1, 1, 700, ("items", "items")),      # five; one shared token
    (3, 32, 8, 1, 1000, 17, ("whole", "items")),     # eight, all rows used, a ragged last page
    (3, 32, 8, 1, 1300, 17, ("items", "items")),
    (2, 11, 6, 2, 4096, 65, ("items", "items")),     # 256 shared pages, the longest context of single waves
    (2, 11, 6, 2, 4097, 65, ((22, 12), (22, 12))),   # one more
    (1, 12, 3, 1, 20000, 30, ((63, 20), (63, 20))),  # slices of eight pages would be more than 64, of 16 more than two rounds of the merge
    (1, 20, 8, 2, 9999, 5, ((40, 16), (40, 16))),    # five row blocks
    (4, 24, 8, 1, 6007, 130, ((32, 12), (32, 12))),  # six; 128 workgroups
    (2, 9, 4, 1, 2500, 7000, ("items", (10, 16))),   # own pages of k_decode_wide in longer slices
    (1, 22, 2, 4, 13072, 200, ((30, 28), (26, 32))),
    (3, 20, 4, 8, 6320, 100, ((10, 40), (5, 80))),   # a workgroup for every unit at dimension 64, half of them at 128
    (12, 19, 4, 2, 11129, 440, ((10, 72), (10, 72))),   # 128 pages would be too many workgroups: of one length for every unit
    (12, 14, 5, 1, 3849, 1181, ("items", (7, 36))),  # as many as fit beside the own pages
    (1, 29, 6, 8, 936, 574, ("whole", (8, 8))),      # all at once in the shorter slices
])
def test_wide_groups_in_every_kind_of_slice(groups, nb, group, hkv, shared, own, want, d):
    hq = hkv * group
    st = dags.decode_state(nb + shared + d, groups, nb, shared, 1, hq, hkv, d,
                           branch_len_list=[1 + (own - 1) * (r % 3) // 2 for r in range(groups * nb)])
    pages = st["desc"]["shared_pages"]
    st["k_pool"][torch.from_numpy(np.ascontiguousarray(pages[len(pages) // 2:])).long()] *= 4.0   # references that are left behind
    dd = B.DecodeDesc(st["desc"], DEV)
    plan = decode_rules.decode(dd.c, hq, hkv, d)
    assert (plan.route if plan.route != "wide" else (plan.splits_a, plan.chunk_a)) == want[d // 128]
    q, out = st["q"].to(DEV), torch.full_like(st["q"], float("nan"), device=DEV)
    ws = torch.empty(B.dag_decode_workspace_bytes(dd, hq, hkv, d), dtype=torch.uint8, device=DEV)
    B.dag_attn_decode(dd, q, st["k_pool"].to(DEV), st["v_pool"].to(DEV), out, ws)
    torch.cuda.synchronize()
    rows = sorted({0, nb - 1, (groups - 1) * nb, groups * nb - 1, groups * nb // 2})
    ref = orc.attn_decode(st["desc"], dags.to_f64(st["q"]), dags.to_f64(st["k_pool"]), dags.to_f64(st["v_pool"]), branches=rows)
    check_close(out[rows], ref[rows], torch.bfloat16, "%d groups x %d branches x %d heads" % (groups, nb, group))
    assert torch.isfinite(out.float()).all()


# Leaves under segments of several lengths: pages of the longest segment's slices, which say what length was chosen (8 pages up to 128), and
# of the others'.  A segment's slices have one length, from 32 pages on an eighth more if that saves one.
@pytest.mark.gpu
@pytest.mark.parametrize("hkv,group,d,sizes,leaves,want", [
    (1, 4, 128, [16 * 10, 16 * 11, 1], [3, 40], [6, 6, None, 2, 4]),                                   # 8 pages: 10 in two slices; nobody reads the third
    (2, 3, 64, [16 * 18, 16 * 19, 300, 16 * 73 - 7], [17, 700, 33], [6, 8, 8, None, 2, 8, 4]),         # 8
    (4, 5, 128, [16 * 320, 16 * 73, 16 * 37, 5], [16 * 18, 16 * 20 + 1, 600], [8, 8, 8, None, 6, 8, 8]),        # 2,028 pages: 8
    (4, 5, 128, [16 * 330, 16 * 73, 16 * 37, 5], [16 * 18, 16 * 20 + 1, 600], [16, 16, 14, None, 10, 12, 14]),  # 2,068: 16
    (8, 2, 128, [16 * 96, 16 * 33], [16 * 40] * 8, [8, 8, 8]),                   # 3,592, no segment longer than 96: 8
    (8, 2, 128, [16 * 97, 16 * 33], [16 * 40] * 8, [14, 12, 14]),                # a longer one: 16
    (8, 4, 128, [16 * 200, 16 * 36 - 3, 16 * 40], [100] * 9, [16, 12, 14, 8]),   # 4,312: 16
    (8, 4, 128, [16 * 258, 16 * 130 - 5, 16 * 65], [16 * 80, 1] * 6, [34, 34, 34, 28, 2]),             # 9,576: 32, and 34 in slices that it saves
    (8, 8, 128, [16 * 145, 16 * 130, 16 * 258], [16 * 145, 16 * 65 + 3] * 24, [50, 66, 66, 50, 66]),   # 71,008: 64
    (8, 1, 64, [16 * 300], [16] * 130, [60, 2]),             # 6,520, but 16 would be 2,600 partials in a room for 780, 32 1,300
    (8, 1, 64, [16 * 361], [16] * 130, [122, 2]),            # 64 would be 910, which the scan finds
    (1, 1, 64, [16 * 5], [7, 33] * 550, [6, 2, 4]),          # more segments than the list's threads
    (1, 1, 64, [16 * 200, 16 * 40], [16 * 9 + 1] * 1100, [68, 40, 10]),   # and partials that are counted first
])
def test_frontiers_in_slices_of_every_length(hkv, group, d, sizes, leaves, want):
    n, m = len(sizes), len(leaves)
    parents = [[i - 1] if i else [] for i in range(n)] + [[i % n] for i in range(m)]  # a chain with leaves at every node of it
    dag = (np.asarray(sizes + leaves, dtype=np.int32), dags.bits_from_sets(dags.closure_from_parents(parents)))
    hq = hkv * group
    st = dags.decode_segments_state(m + d + group, [dag], [list(range(n, n + m))], hq, hkv, d, keep_tokens=False)
    sd = B.SegDecodeDesc(st["desc"], DEV)
    out = torch.full_like(st["q"], float("nan"), device=DEV)
    ws = torch.empty(B.dag_decode_segments_workspace_bytes(sd, hq, hkv, d), dtype=torch.uint8, device=DEV).fill_(0xff)
    B.dag_attn_decode_segments(sd, st["q"].to(DEV), st["k_pool"].to(DEV), st["v_pool"].to(DEV), out, ws)
    torch.cuda.synchronize()
    slices = decode_rules.listed_slices(decode_rules.segments(sd.c, hq, hkv, d), ws.cpu().numpy())
    assert [slices.get((int(st["desc"]["seg_page_off"][s]), 0)) for s in range(len(want))] == want
    rows = list(range(m)) if m < 24 else sorted({0, 1, m // 2, m - 2, m - 1})
    ref = orc.attn_decode_segments(st["desc"], dags.to_f64(st["q"]), dags.to_f64(st["k_pool"]), dags.to_f64(st["v_pool"]), branches=rows)
    check_close(out[rows], ref[rows], torch.bfloat16, "frontier of %d leaves" % m)
    assert torch.isfinite(out.float()).all()
