"""GPU parity of dag_attn_decode with many sibling groups, empty ones among them: the group of a branch is looked up 64
groups at a time."""
import numpy as np
import pytest
import torch

from oracle import dag_oracle as orc
from workloads import dags
from tests.gpu_util import check_close
from tests.test_gpu_decode import _gpu_decode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_groups", [1, 2, 63, 64, 65, 128, 129, 4096, 4097])
def test_many_groups(n_groups):
    hq, hkv, d = 4, 2, 64
    rng = np.random.Generator(np.random.PCG64(n_groups))
    st = dags.decode_state(70 + n_groups, n_seqs=n_groups, n_branches=2, shared_len=17, branch_len=0, hq=hq, hkv=hkv, d=d,
                           branch_len_list=rng.integers(1, 20, 2 * n_groups))
    off = st["desc"]["group_branch_off"].copy()
    for g in range(2, n_groups, 3):      # every third group hands its branches to the one in front (the first and the last group too)
        off[g] = off[g + 1]
    if n_groups > 2:
        off[1] = 0
        off[n_groups - 1] = off[n_groups]
    st["desc"]["group_branch_off"] = off
    out, kp, vp = _gpu_decode(st, hq, hkv, d, 1e4)
    rows = np.unique(np.concatenate([[0, 1, 2 * n_groups - 2, 2 * n_groups - 1], rng.integers(0, 2 * n_groups, 60)]))
    ref = orc.attn_decode(st["desc"], dags.to_f64(st["q"]), dags.to_f64(kp), dags.to_f64(vp), branches=rows)
    check_close(out[rows], ref[rows], torch.bfloat16, "%d groups" % n_groups)


# 4096 rows (branches x heads) take the merge of few rows, 4128 and 4160 that of many; 2, 6 and 17 partials to a row
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("groups,branches,hkv,shared,own", [(32, 4, 8, 17, 9), (43, 3, 8, 17, 9), (43, 3, 2, 2500, 200), (10, 13, 1, 12000, 700)])
def test_merge_of_few_and_of_many_rows(groups, branches, hkv, shared, own, d):
    hq, n = 32, groups * branches
    st = dags.decode_state(900 + n + d, groups, branches, shared, 1, hq, hkv, d, branch_len_list=[max(1, own - 40 * (r % 5)) for r in range(n)])
    out, kp, vp = _gpu_decode(st, hq, hkv, d, 1e4)
    rows = np.array([0, 1, n // 2, n - 2, n - 1])
    ref = orc.attn_decode(st["desc"], dags.to_f64(st["q"]), dags.to_f64(kp), dags.to_f64(vp), branches=rows)
    check_close(out[rows], ref[rows], torch.bfloat16, "%d rows" % (n * hq))
