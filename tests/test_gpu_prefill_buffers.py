"""GPU: dag_attn_prefill with buffers that overlap or are shared between calls in the ways it takes them: the output
on the memory of V or Q, and workspaces prepared once for several head counts."""
import numpy as np
import pytest
import torch

from paper_2602_07529_amd import binding as B
from workloads import dags
from tests.gpu_util import DEV, build_meta

pytestmark = pytest.mark.gpu


def _batch(hq, hkv, d):
    # many chunks for every compute unit: rows are written while others still read
    dag_list = [dags.fork_join(1024, [256] * 6, 320), dags.fork_join(700, [130, 260, 90], 200)] * 2
    T = int(sum(int(np.sum(L)) for L, _ in dag_list))
    q, k, v = (x.to(DEV) for x in dags.make_qkv(300 + hq, T, hq, hkv, d, 0.5, torch.bfloat16))
    return q, k, v, build_meta(dag_list, hq, hkv, d, torch.bfloat16)[1]


def _close(got, ref):
    # two correct orders of the keys: bf16 probabilities and results
    assert torch.isfinite(got.float()).all()
    assert float((got.double() - ref.double()).norm()) <= 1e-2 * float(ref.double().norm())


@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("hq,hkv,d", [(8, 8, 128), (16, 16, 64), (16, 8, 128)])
def test_output_on_the_memory_of_v(hq, hkv, d, prepared):
    q, k, v, meta = _batch(hq, hkv, d)
    ref = torch.empty_like(q)
    B.dag_attn_prefill(meta, q, k, v, ref)
    ws = torch.empty(B.dag_prefill_workspace_bytes(meta, hkv, d, B.DAG_BF16), dtype=torch.uint8, device=DEV)
    if prepared:
        B.dag_prefill_prepare_v(meta, v, hq, workspace=ws)
        again = torch.empty_like(q)
        B.dag_attn_prefill(meta, q, k, v, again, workspace=ws, prepared=True)
        assert torch.equal(again, ref)
    memory = torch.empty(q.numel(), dtype=q.dtype, device=DEV)
    v_in = memory[-v.numel():].view_as(v)   # (hq > hkv: on the last rows of the output)
    v_in.copy_(v)
    out = memory.view_as(q)
    B.dag_attn_prefill(meta, q, k, v_in, out, workspace=ws, prepared=prepared)
    _close(out, ref)
    if prepared:   # and the workspace is what it was
        B.dag_attn_prefill(meta, q, k, v, again, workspace=ws, prepared=True)
        assert torch.equal(again, ref)


@pytest.mark.parametrize("hq,hkv,d", [(32, 8, 128), (8, 8, 64)])
def test_output_on_the_memory_of_q(hq, hkv, d):
    q, k, v, meta = _batch(hq, hkv, d)
    ref = torch.empty_like(q)
    B.dag_attn_prefill(meta, q, k, v, ref)
    B.dag_attn_prefill(meta, q, k, v, q)
    assert torch.equal(q, ref)


# the grouping the workspace was prepared for, the one it is used with: every launch shape finds its tables
@pytest.mark.parametrize("first,then", [(4, 8), (8, 4), (6, 2), (1, 5), (7, 3), (4, 2), (5, 7)])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("small", [False, True])
def test_prepared_for_another_head_count(first, then, d, small):
    hkv = 2
    dag_list = [dags.fork_join(130, [40, 64, 33, 150, 63], 70)] * (1 if small else 30)
    T = int(sum(int(np.sum(L)) for L, _ in dag_list))
    q, k, v = (x.to(DEV) for x in dags.make_qkv(310 + then, T, then * hkv, hkv, d, 0.5, torch.bfloat16))
    _, meta = build_meta(dag_list, then * hkv, hkv, d, torch.bfloat16)
    ref, out = torch.empty_like(q), torch.empty_like(q)
    B.dag_attn_prefill(meta, q, k, v, ref)
    ws = torch.zeros(B.dag_prefill_workspace_bytes(meta, hkv, d, B.DAG_BF16), dtype=torch.uint8, device=DEV)
    B.dag_prefill_prepare_v(meta, v, first * hkv, workspace=ws)
    B.dag_attn_prefill(meta, q, k, v, out, workspace=ws, prepared=True)
    assert torch.equal(out, ref)
