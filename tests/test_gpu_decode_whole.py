"""Decode steps over short contexts, which one workgroup per (branch, KV head) takes whole, and their neighbours that items and a merge take."""
import pytest
import torch

from oracle import dag_oracle as orc
from paper_2602_07529_amd import binding as B
from workloads import dags
from tests import decode_rules
from tests.gpu_util import DEV, check_close


# groups, branches, heads per KV head, KV heads, head dimension, shared tokens, longest own context, route.  The bound is that of every
# decode test.
@pytest.mark.gpu
@pytest.mark.parametrize("groups,nb,group,hkv,d,shared,own,route", [
    (1, 1, 1, 1, 128, 1, 1, "whole"),          # seven of eight waves with nothing or one token
    (1, 4, 8, 2, 128, 512, 320, "whole"),      # 32 + 20 pages: the longest of one row block at this dimension
    (1, 4, 8, 2, 128, 512, 321, "items"),      # a page more
    (1, 5, 8, 2, 128, 992, 32, "whole"),       # two row blocks, 62 + 2 pages: the longest
    (1, 5, 8, 2, 128, 993, 32, "items"),       # a page more
    (2, 3, 4, 2, 64, 17, 16 * 94, "whole"),    # 2 + 94 pages, nearly all of them own ones
    (2, 3, 4, 2, 64, 33, 16 * 94, "items"),    # a page more
    (3, 5, 5, 8, 128, 499, 299, "whole"),      # odd numbers of pages, ragged last ones
    (3, 5, 5, 2, 128, 499, 331, "items"),
    (2, 7, 9, 1, 128, 100, 40, "items"),       # nine rows a branch
    (70, 1, 3, 1, 64, 45, 20, "whole"),        # more groups than a wave has lanes
    (2, 32, 7, 4, 128, 200, 50, "whole"),      # 256 workgroups
    (1, 257, 1, 1, 64, 60, 20, "items"),       # 257; groups of more than 32 rows
])
def test_short_contexts(groups, nb, group, hkv, d, shared, own, route):
    hq, live = hkv * group, groups * nb
    st = dags.decode_state(nb + shared + d, groups, nb, shared, 1, hq, hkv, d, branch_len_list=[1 + (own - 1) * ((r + 2) % 3) // 2 for r in range(live)])
    dd = B.DecodeDesc(st["desc"], DEV)
    assert decode_rules.decode(dd.c, hq, hkv, d).route == route
    q, k, v = (st[x].to(DEV) for x in ("q", "k_pool", "v_pool"))
    ws = torch.full((B.dag_decode_workspace_bytes(dd, hq, hkv, d),), 0xff, dtype=torch.uint8, device=DEV)
    out, again = (torch.full_like(st["q"], float("nan"), device=DEV) for _ in range(2))
    B.dag_attn_decode(dd, q, k, v, out, ws)
    B.dag_attn_decode(dd, q, k, v, again, ws)
    torch.cuda.synchronize()
    assert torch.equal(out, again) and torch.isfinite(out.float()).all()
    rows = sorted({0, nb - 1, live - nb, live - 1, live // 2})
    ref = orc.attn_decode(st["desc"], dags.to_f64(st["q"]), dags.to_f64(st["k_pool"]), dags.to_f64(st["v_pool"]), branches=rows)
    check_close(out[rows], ref[rows], torch.bfloat16, "%d groups x %d branches x %d heads" % (groups, nb, group))
