"""GPU: dK / dV whose streams of query rows are cut into pieces, against the fp64 oracle: pieces of whole and of
masked tiles, pairs of one piece beside pairs of many, keys that end inside a pair, hidden values in one piece."""
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
    rng = np.random.Generator(np.random.PCG64(7100))
    return {
        "fork": [dags.fork_join(701, [90, 64, 131] * 4, 230), dags.linear_chain([30, 40])],
        "random": [dags.random_dag(rng, n_nodes=70, depth=5, len_lo=10, len_hi=60)[:2] for _ in range(2)],
        "chain": [dags.linear_chain([2049])],
    }[name]


def _without_pieces(meta, hq, hkv, d):
    up = lambda n: -(-n // 256) * 256  # noqa: E731
    m = meta.sizes
    n = 2 * up(m.total_tokens * hq * 4) + 2 * up(m.total_ktiles * 4) + up(m.total_tokens * 8) + 256
    if hq // hkv % (4 if d == 128 else 2):
        n += up(m.total_tiles * 4) + up(m.total_tiles) + 3 * up(m.total_qtiles * 4 + 4)
    return n


@pytest.mark.parametrize("name", ["fork", "random", "chain"])
@pytest.mark.parametrize("hq,hkv,d", [(1, 1, 64), (5, 1, 64), (4, 2, 64), (1, 1, 128), (6, 1, 128), (8, 2, 128)])
@pytest.mark.parametrize("pieces", [True, False])
def test_dkv_in_pieces(name, hq, hkv, d, pieces, monkeypatch):
    dag_list = _dags(name)
    _, meta = build_meta(dag_list, hq, hkv, d, torch.bfloat16)
    small = _without_pieces(meta, hq, hkv, d)
    assert small < B.dag_prefill_bwd_workspace_bytes(meta, hq, hkv, d)
    if not pieces:   # a workspace without room for them is taken
        call = B.dag_attn_prefill_bwd
        monkeypatch.setattr(B, "dag_attn_prefill_bwd", lambda m, q, *args, **kw: call(
            m, q, *args, workspace=torch.empty(small, dtype=torch.uint8, device=q.device), **kw))
    inputs, grads = _forward_backward(dag_list, hq, hkv, d, 7200 + hq)
    _check_against_oracle(dag_list, inputs, grads)


@pytest.mark.parametrize("hq,hkv,d", [(2, 1, 64), (3, 1, 128)])
def test_hidden_rows_in_one_piece(hq, hkv, d):
    """A branch of Inf: its rows share tiles with rows that see the keys of the first branch, in one piece of several."""
    dag_list = [dags.fork_join(50, [1000, 130, 900], 400)]
    L, anc = dag_list[0]
    T = int(np.sum(L))
    q, k, v = dags.make_qkv(7300, T, hq, hkv, d, 0.7, torch.bfloat16)
    dout = dags.make_qkv(7301, T, hq, hkv, d, 1.0, torch.bfloat16)[0]
    ref = orc.attn_prefill_bwd(*(dags.to_f64(x) for x in (q, k, v, dout)), L, anc)
    _, meta = build_meta(dag_list, hq, hkv, d, torch.bfloat16)
    out, lse = torch.empty_like(q, device=DEV), torch.empty(T, hq, dtype=torch.float32, device=DEV)
    B.dag_attn_prefill(meta, q.to(DEV), k.to(DEV), v.to(DEV), out, lse)
    # rows 1050 .. 1179 are hidden from the keys of nodes 1 and 3, whose other rows lie around them
    bad = slice(1050, 1180)
    qd, dod = q.to(DEV), dout.to(DEV)
    qd[bad], dod[bad] = float("inf"), float("inf")
    dq, dk, dv = torch.empty_like(qd), torch.empty(T, hkv, d, dtype=torch.bfloat16, device=DEV), torch.empty(T, hkv, d, dtype=torch.bfloat16, device=DEV)
    B.dag_attn_prefill_bwd(meta, qd, k.to(DEV), v.to(DEV), out, dod, lse, dq, dk, dv)
    torch.cuda.synchronize()
    for sl in (slice(50, 1050), slice(1180, T)):
        check_close(dk[sl], ref[1][sl], torch.bfloat16, "dk")
        check_close(dv[sl], ref[2][sl], torch.bfloat16, "dv")
    assert not torch.isfinite(dv[:50].float()).all(dim=-1).any()
