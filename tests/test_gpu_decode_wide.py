"""Wide sibling groups: the pipeline over the shared pages at every number of row blocks (one wave, two waves, four waves to
a block), at the ends of its tiles of 64 tokens, and with scores that leave the range of the reference maximum."""
import numpy as np
import pytest
import torch

from oracle import dag_oracle as orc
from paper_2602_07529_amd import binding as B
from workloads import dags
from tests import decode_rules
from tests.gpu_util import DEV, check_close

pytestmark = pytest.mark.gpu


# 32 groups x 8 KV heads: a workgroup has the whole shared list of a group, 128 pages at most.  Own contexts of a token to three; of 94 to
# 96 where the shared lists are so little work that single waves would take them.
@pytest.mark.parametrize("nb,group,shared,own", [
    (9, 4, 2048, 3), (9, 4, 2001, 3), (9, 4, 63, 3),     # two row blocks, two waves each: 32 tiles; 31 and a ragged one; single waves
    (12, 6, 129, 3), (12, 6, 192, 3),                    # three: an even number of tiles and a token; an odd number; at dimension 64 single waves
    (16, 8, 64, 3), (16, 8, 1024, 3), (16, 8, 1087, 3),  # four, all rows used; the first by single waves
    (20, 8, 64, 3), (20, 8, 65, 3), (20, 8, 2048, 3),    # five: the last one over four waves; the first, at dimension 64 the second, by single waves
    (23, 8, 128, 3), (23, 8, 1999, 3),                   # six: the last two over two waves each, partly filled
    (28, 8, 191, 3), (32, 8, 1, 3), (32, 8, 2032, 3),    # seven and eight, a wave each; one token at dimension 64 by single waves
    (9, 4, 63, 96), (12, 6, 129, 96), (12, 6, 192, 96),  # no whole tile; and the short ones above, by the wide kernel
    (16, 8, 64, 96), (20, 8, 64, 96), (20, 8, 65, 96), (32, 8, 1, 96),
])
@pytest.mark.parametrize("d,growth", [(128, 1.0), (64, 8.0)])
def test_wide_groups_at_every_number_of_row_blocks(nb, group, shared, own, d, growth):
    hkv, groups, head, g = 8, 32, 5, 17
    hq = hkv * group
    st = dags.decode_state(nb + shared, groups, nb, shared, 1, hq, hkv, d, branch_len_list=[own - 2 + r % 3 for r in range(groups * nb)])
    desc = st["desc"]
    for g0 in range(groups):  # keys of the later pages have `growth` times the scores of the earlier ones
        pages = desc["shared_pages"][desc["shared_page_off"][g0]:desc["shared_page_off"][g0 + 1]]
        st["k_pool"][torch.from_numpy(np.ascontiguousarray(pages[len(pages) // 3:])).long()] *= growth
    dd = B.DecodeDesc(desc, DEV)
    narrow = own < 16 and -(-nb * group // 32) * -(-shared // 16) * d <= 22 * 128 and nb * d <= 25 * 128   # 5632 shared and 6400 own pages in all
    assert decode_rules.decode(dd.c, hq, hkv, d).route == ("items" if narrow else "wide")
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


# Probabilities are rounded to 16 bits relative to a reference maximum, and those just below a power of two, where the largest are
# when the reference is their maximum, lose the least.  So the references have to stay near it: the error against 64 bits, as a
# part of what probabilities relative to the row's maximum give, is 0.911, 0.930, 0.908, 0.928, 0.945 and 0.911, 0.945, 0.979 here.  In single waves
# and in a workgroup to a branch the reference is the running maximum; in wide groups it is that of the first 64 keys of a shared slice, raised when
# a lane's sum grows by 3 or 2.5 in slices longer than the workspace is sized for (not in the fifth row), and the running one in the own pages.
# With references that may be exceeded by 2^8 in own pages and single waves, and by sums of 1024 in shared slices: 0.984, 1.001, 0.983, 0.948, 0.971 and
# 0.944, 0.980, 1.013.  `most` lies between.  (The first three rows were wide groups once, with 0.910, 0.925, 0.902.)
@pytest.mark.parametrize("groups,nb,shared,own,hq,hkv,d,most,route", [
    (10, 10, 2021, 114, 8, 2, 64, 0.93, "items"), (4, 22, 526, 80, 2, 1, 128, 0.945, "whole"), (6, 8, 3760, 258, 16, 2, 64, 0.925, "items"),
    (10, 15, 141, 885, 5, 1, 128, 0.965, "wide"), (15, 29, 104, 234, 10, 2, 128, 0.99, "wide"),
    (4, 22, 4526, 80, 2, 1, 128, 0.927, "wide"), (6, 8, 4760, 258, 16, 2, 64, 0.963, "wide"), (16, 20, 1900, 300, 16, 8, 128, 0.997, "wide")])
def test_probabilities_are_rounded_near_the_maximum(groups, nb, shared, own, hq, hkv, d, most, route):
    st = dags.decode_state(11, groups, nb, shared, own, hq, hkv, d)
    dd = B.DecodeDesc(st["desc"], DEV)
    assert decode_rules.decode(dd.c, hq, hkv, d).route == route
    q, out = st["q"].to(DEV), torch.empty_like(st["q"], device=DEV)
    ws = torch.empty(B.dag_decode_workspace_bytes(dd, hq, hkv, d), dtype=torch.uint8, device=DEV)
    B.dag_attn_decode(dd, q, st["k_pool"].to(DEV), st["v_pool"].to(DEV), out, ws)
    torch.cuda.synchronize()
    bf16 = lambda x: x.to(torch.bfloat16).double()  # noqa: E731
    err = err_ref = 0.0
    kp, vp = dags.to_f64(st["k_pool"]), dags.to_f64(st["v_pool"])
    for r in range(0, groups * nb, max(1, groups * nb // 48)):
        for h in range(hkv):
            k, v = (torch.from_numpy(np.ascontiguousarray(x)) for x in orc.gather_context(st["desc"], r, h, kp, vp))
            rows = slice(h * hq // hkv, (h + 1) * hq // hkv)
            s = st["q"][r, rows].double() @ k.T / d ** 0.5
            p = torch.exp(s - s.max(dim=-1, keepdim=True).values)
            total = p.sum(dim=-1, keepdim=True)
            exact = p @ v / total
            err += (out[r, rows].cpu().double() - exact).square().sum().item()
            err_ref += (bf16(bf16(p) @ v / total) - exact).square().sum().item()
    assert err < most ** 2 * err_ref, "%.4f of the error with the row's maximum" % (err / err_ref) ** 0.5


@pytest.mark.parametrize("groups,nb,shared,hq,hkv,d", [(2, 32, 16000, 16, 4, 64), (1, 12, 30000, 24, 8, 128)])
def test_equal_scores_take_no_longer(groups, nb, shared, hq, hkv, d):
    """Keys of zeros make every score equal: no probability leaves the reference.  Against keys that are largest in the first eight
    pages of every slice, where the reference comes from, so that every other probability is next to nothing: the same launch,
    the same time (of the two runs of one kind, the shortest of twelve, differ by less than 2 %)."""
    st = dags.decode_state(5, groups, nb, shared, 1, hq, hkv, d, branch_len_list=[1] * (groups * nb))
    plan = decode_rules.decode(B.DecodeDesc(st["desc"], DEV).c, hq, hkv, d)
    assert plan.route == "wide" and plan.settle < 1024   # slices longer than the workspace is sized for
    q, dd = torch.ones_like(st["q"], device=DEV), B.DecodeDesc(st["desc"], DEV)
    out, vp = torch.empty_like(q), st["v_pool"].to(DEV)
    equal = torch.zeros_like(st["k_pool"], device=DEV)
    first = equal.clone()
    for g in range(groups):
        pages = st["desc"]["shared_pages"][st["desc"]["shared_page_off"][g]:st["desc"]["shared_page_off"][g + 1]]
        lead = np.concatenate([pages[i:i + 8] for i in range(0, len(pages), plan.chunk_a)])
        first[torch.from_numpy(lead).long().to(DEV)] = 2.0
    ws = torch.empty(B.dag_decode_workspace_bytes(dd, hq, hkv, d), dtype=torch.uint8, device=DEV)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = [float("inf")] * 2
    for turn in range(24):
        kp = (equal, first)[turn % 2]
        for _ in range(3):
            B.dag_attn_decode(dd, q, kp, vp, out, ws)
        a.record()
        for _ in range(30):
            B.dag_attn_decode(dd, q, kp, vp, out, ws)
        b.record()
        torch.cuda.synchronize()
        best[turn % 2] = min(best[turn % 2], a.elapsed_time(b) / 30)
    assert best[0] < 1.1 * best[1], "%.1f us with equal scores, %.1f us without" % (best[0] * 1e3, best[1] * 1e3)
