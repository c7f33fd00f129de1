"""Sibling groups of more than 32 rows of a KV head: single-wave items where little is to be read, longer slices of the shared pages
elsewhere; and the workspace, whose size follows the shorter slices whatever the launch takes."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import dag_oracle as orc
from paper_2602_07529_amd import binding as B
from workloads import dags
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


# groups, branches, heads per KV head, KV heads, shared tokens, longest own context.  The error bound is that of every decode test.
@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("groups,nb,group,hkv,shared,own", [
    (2, 9, 4, 1, 33, 3),        # single waves: two row blocks, the second with four rows
    (1, 13, 5, 2, 1, 40),       # three; one shared token
    (3, 32, 8, 1, 1000, 17),    # eight, all rows used, a ragged last page
    (2, 11, 6, 2, 4096, 65),    # 256 shared pages, the longest context of single waves
    (2, 11, 6, 2, 4097, 65),    # one more: slices of 52 pages and a page
    (1, 12, 3, 1, 20000, 30),   # longer slices, 128 of which would leave 98 pages to the last: of one length
    (1, 20, 8, 2, 9999, 5),     # five row blocks
    (4, 24, 8, 1, 6007, 130),   # six
    (2, 9, 4, 1, 2500, 7000),   # own pages of k_decode_wide in longer slices
])
def test_wide_groups_in_every_kind_of_slice(groups, nb, group, hkv, shared, own, d):
    hq = hkv * group
    st = dags.decode_state(nb + shared + d, groups, nb, shared, 1, hq, hkv, d,
                           branch_len_list=[1 + (own - 1) * (r % 3) // 2 for r in range(groups * nb)])
    pages = st["desc"]["shared_pages"]
    st["k_pool"][torch.from_numpy(np.ascontiguousarray(pages[len(pages) // 2:])).long()] *= 4.0   # references that are left behind
    dd = B.DecodeDesc(st["desc"], DEV)
    q, out = st["q"].to(DEV), torch.full_like(st["q"], float("nan"), device=DEV)
    ws = torch.empty(B.dag_decode_workspace_bytes(dd, hq, hkv, d), dtype=torch.uint8, device=DEV)
    B.dag_attn_decode(dd, q, st["k_pool"].to(DEV), st["v_pool"].to(DEV), out, ws)
    torch.cuda.synchronize()
    rows = sorted({0, nb - 1, (groups - 1) * nb, groups * nb - 1, groups * nb // 2})
    ref = orc.attn_decode(st["desc"], dags.to_f64(st["q"]), dags.to_f64(st["k_pool"]), dags.to_f64(st["v_pool"]), branches=rows)
    check_close(out[rows], ref[rows], torch.bfloat16, "%d groups x %d branches x %d heads" % (groups, nb, group))
    assert torch.isfinite(out.float()).all()


# Leaves under segments of several lengths: the slices that the pages to be read call for (8 pages up to 128, for these shapes by name),
# segments whose last pages join a slice (65 of 64 pages, 130 of 128), which do not (73, 145), of one page and of one token.
@pytest.mark.gpu
@pytest.mark.parametrize("hkv,group,d,sizes,leaves", [
    (1, 4, 128, [16 * 10, 16 * 11, 1], [3, 40]),                                # 8 pages: 10 in one slice, 11 in two
    (2, 3, 64, [16 * 18, 16 * 19, 300, 16 * 73 - 7], [17, 700, 33]),            # 8
    (2, 5, 128, [16 * 300, 16 * 73, 16 * 37, 5], [16 * 18, 16 * 20 + 1, 600]),  # 16
    (8, 4, 128, [16 * 200, 16 * 36 - 3, 16 * 40], [100] * 9),                   # 32: two row blocks
    (8, 8, 128, [16 * 258, 16 * 130 - 5, 16 * 65], [16 * 66, 1] * 6),           # 64: three row blocks
    (8, 8, 128, [16 * 145, 16 * 130, 16 * 258], [16 * 145, 16 * 65 + 3] * 12),  # 128: six
])
def test_frontiers_in_slices_of_every_length(hkv, group, d, sizes, leaves):
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
    ref = orc.attn_decode_segments(st["desc"], dags.to_f64(st["q"]), dags.to_f64(st["k_pool"]), dags.to_f64(st["v_pool"]))
    check_close(out, ref, torch.bfloat16, "frontier of %d leaves" % m)
