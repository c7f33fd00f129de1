"""GPU: dK / dV on blocks of keys that are cut at node borders, against the fp64 oracle: blocks of one node and of several, of 64 to
128 keys and shorter ones at the end, sequences that keep blocks of 128 beside others, one and two visibility words."""
import numpy as np
import pytest
import torch

from oracle import dag_oracle as orc
from paper_2602_07529_amd import binding as B
from workloads import dags
from tests.gpu_util import DEV, build_meta
from tests.test_gpu_prefill_bwd import _check_against_oracle, _forward_backward, check_close

pytestmark = pytest.mark.gpu


def _dags(name):
    rng = np.random.Generator(np.random.PCG64(8100))
    return {
        # every block ends at a border (64, 65, 127, 128 and 129 keys a node), last blocks of 1 and of 63 keys
        "edges": [dags.linear_chain([64, 65, 127, 128, 129, 1, 63, 192] * 3 + [1]), dags.fork_join(700, [128, 64, 129, 127, 1] * 2, 63),
                  dags.linear_chain([133])],
        "words": [dags.random_dag(rng, n_nodes=100, depth=6, len_lo=1, len_hi=60)[:2], dags.random_dag(rng, n_nodes=64, depth=5, len_lo=20, len_hi=60)[:2]],
        # siblings of about 100 tokens, for which blocks of 128 keys cost less, beside one that is cut
        "even": [dags.fork_join(484, [106, 90, 120, 100] * 2, 229), dags.random_dag(rng, n_nodes=40, depth=5, len_lo=30, len_hi=150)[:2], dags.linear_chain([700])],
    }[name]


@pytest.mark.parametrize("name", ["edges", "words", "even"])
@pytest.mark.parametrize("hq,hkv,d", [(2, 1, 64), (8, 2, 64), (4, 2, 128), (5, 1, 128)])
def test_dkv_blocks(name, hq, hkv, d):
    dag_list = _dags(name)
    assert sum(int(np.sum(L)) for L, _ in dag_list) >= 4096
    inputs, grads = _forward_backward(dag_list, hq, hkv, d, 8200 + hq)
    _check_against_oracle(dag_list, inputs, grads)


@pytest.mark.parametrize("hq,hkv,d", [(2, 1, 64), (3, 1, 128)])
def test_hidden_keys_behind_a_short_block(hq, hkv, d):
    """A branch whose rows are Inf, next to blocks of fewer than 128 keys: the lanes of those blocks without a key of their own take part
    in the tiles without masks and must not reach anything that is stored."""
    L, anc = dag = dags.fork_join(50, [1000, 130, 900, 70, 1900], 300)
    T = int(np.sum(L))
    assert T >= 4096
    q, k, v = dags.make_qkv(8300, T, hq, hkv, d, 0.7, torch.bfloat16)
    dout = dags.make_qkv(8301, T, hq, hkv, d, 1.0, torch.bfloat16)[0]
    ref = orc.attn_prefill_bwd(*(dags.to_f64(x) for x in (q, k, v, dout)), L, anc)
    _, meta = build_meta([dag], hq, hkv, d, torch.bfloat16)
    out, lse = torch.empty_like(q, device=DEV), torch.empty(T, hq, dtype=torch.float32, device=DEV)
    B.dag_attn_prefill(meta, q.to(DEV), k.to(DEV), v.to(DEV), out, lse)
    bad = slice(1050, 1180)  # the second branch
    qd, dod = q.to(DEV), dout.to(DEV)
    qd[bad], dod[bad] = float("inf"), float("inf")
    dq, dk, dv = torch.empty_like(qd), torch.empty(T, hkv, d, dtype=torch.bfloat16, device=DEV), torch.empty(T, hkv, d, dtype=torch.bfloat16, device=DEV)
    B.dag_attn_prefill_bwd(meta, qd, k.to(DEV), v.to(DEV), out, dod, lse, dq, dk, dv)
    torch.cuda.synchronize()
    for sl in (slice(50, 1050), slice(1180, T)):
        check_close(dk[sl], ref[1][sl], torch.bfloat16, "dk")
        check_close(dv[sl], ref[2][sl], torch.bfloat16, "dv")
    assert not torch.isfinite(dv[:50].float()).all(dim=-1).any()
