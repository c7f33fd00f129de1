"""Wide sibling groups: the pipeline over the shared pages at every number of row blocks (one wave, two waves, four waves to
a block), at the ends of its tiles of 64 tokens, and with scores that leave the range of the reference maximum."""
import numpy as np
import pytest
import torch

from oracle import dag_oracle as orc
from paper_2602_07529_amd import binding as B
from workloads import dags
from tests.gpu_util import DEV, check_close

pytestmark = pytest.mark.gpu


# 32 groups x 8 KV heads: a workgroup has the whole shared list of a group, 128 pages at most
@pytest.mark.parametrize("nb,group,shared", [
    (9, 4, 2048), (9, 4, 2001), (9, 4, 63),          # two row blocks, two waves each: 32 tiles; 31 and a ragged one; no whole tile
    (12, 6, 129), (12, 6, 192),                      # three: an even number of tiles and a token; an odd number
    (16, 8, 64), (16, 8, 1024), (16, 8, 1087),       # four, all rows used
    (20, 8, 64), (20, 8, 65), (20, 8, 2048),         # five: the last one over four waves
    (23, 8, 128), (23, 8, 1999),                     # six: the last two over two waves each, partly filled
    (28, 8, 191), (32, 8, 1), (32, 8, 2032),         # seven and eight, a wave each
])
@pytest.mark.parametrize("d,growth", [(128, 1.0), (64, 8.0)])
def test_wide_groups_at_every_number_of_row_blocks(nb, group, shared, d, growth):
    hkv, groups, head, g = 8, 32, 5, 17
    hq = hkv * group
    st = dags.decode_state(nb + shared, groups, nb, shared, 1, hq, hkv, d, branch_len_list=[1 + r % 3 for r in range(groups * nb)])
    desc = st["desc"]
    for g0 in range(groups):  # keys of the later pages have `growth` times the scores of the earlier ones
        pages = desc["shared_pages"][desc["shared_page_off"][g0]:desc["shared_page_off"][g0 + 1]]
        st["k_pool"][torch.from_numpy(np.ascontiguousarray(pages[len(pages) // 3:])).long()] *= growth
    dd = B.DecodeDesc(desc, DEV)
    kp, vp, q = st["k_pool"].to(DEV), st["v_pool"].to(DEV), st["q"].to(DEV)
    out = torch.full_like(q, float("nan"))
    ws = torch.empty(B.dag_decode_workspace_bytes(dd, hq, hkv, d), dtype=torch.uint8, device=DEV)
    B.dag_attn_decode(dd, q, kp, vp, out, ws)
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all()
    # one KV head of one group against the oracle (a pool of that head alone)
    one = dict(desc)
    rows = slice(g * nb, (g + 1) * nb)
    heads = slice(head * group, (head + 1) * group)
    ref = orc.attn_decode(one, dags.to_f64(st["q"][:, heads]), dags.to_f64(st["k_pool"][:, head:head + 1]),
                          dags.to_f64(st["v_pool"][:, head:head + 1]), branches=list(range(g * nb, (g + 1) * nb)))
    check_close(out[rows, heads], ref[rows], torch.bfloat16, "%d branches x %d heads, %d tokens" % (nb, group, shared))
