"""GPU: dQ on query chunks, whose items hold all heads of a group as row-major (row, head) pairs, against the fp64 oracle: groups with pairs
that belong to no row or no head, waves without rows, items of more than eight heads, tiles shared out over several workgroups."""
import numpy as np
import pytest
import torch

from paper_2602_07529_amd import binding as B
from workloads import dags
from tests.gpu_util import DEV, build_meta, launched_kernels
from tests.test_gpu_prefill_bwd import _check_against_oracle, _forward_backward

pytestmark = pytest.mark.gpu


def _dags(name):
    rng = np.random.Generator(np.random.PCG64(8400))
    return {
        # remainders of every chunk size (256 to 16 rows), one token, two visibility words
        "batch": [dags.fork_join(130, [40, 64, 3, 150, 63], 70), dags.linear_chain([1]), dags.linear_chain([65, 190, 257]),
                  dags.random_dag(rng, n_nodes=70, depth=6, len_lo=10, len_hi=40)[:2]],
        # few chunks of many tiles: pieces
        "pieces": [dags.fork_join(1100, [70, 33], 51)],
    }[name]


@pytest.mark.parametrize("name", ["batch", "pieces"])
@pytest.mark.parametrize("g", [1, 2, 3, 4, 5, 7, 8, 9, 17])
@pytest.mark.parametrize("d", [64, 128])
def test_every_group(name, g, d):
    hkv = 2 if name == "batch" and g < 9 else 1
    dag_list = _dags(name)
    inputs, grads = _forward_backward(dag_list, g * hkv, hkv, d, 8500 + g + d)
    _check_against_oracle(dag_list, inputs, grads)


# chunks that nearly fill the device: in pieces only where some may be much longer than the others, and then the long ones
@pytest.mark.parametrize("name,pieces", [("long fork", True), ("short fork", False), ("random", False)])
@pytest.mark.parametrize("hq,hkv,d,rows", [(7, 1, 128, 36), (8, 4, 64, 64)])
def test_pieces_of_chunks_that_fill_the_device(name, pieces, hq, hkv, d, rows):
    rng = np.random.Generator(np.random.PCG64(8600))
    n = {128: 7400, 64: 6200}[d]   # tokens that make about 0.8 of the chunks that go at once
    dag_list = {"long fork": [dags.fork_join(n // 8, [n // 10] * 8, n - n // 8 - n // 10 * 8)],
                "short fork": [dags.fork_join(700, [200] * 3, n // 4 - 1300)] * 4,
                "random": [dags.random_dag(rng, n_nodes=30, depth=5, len_lo=n // 62, len_hi=n // 21)[:2]]}[name]
    T, nodes = sum(int(np.sum(L)) for L, _ in dag_list), sum(len(L) for L, _ in dag_list)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    full = units * (1 if d == 128 else 2)
    assert 4 * (T // rows + nodes // 2) * hkv >= 3 * full and (T // rows + nodes) * hkv <= full
    assert pieces == (sum(-(-int(np.sum(L)) // 64) for L, _ in dag_list) >= 52 * len(dag_list) and T >= 256 * nodes)
    inputs, grads = _forward_backward(dag_list, hq, hkv, d, 8700)
    _, meta = build_meta(dag_list, hq, hkv, d, torch.bfloat16)
    q, k, v, dout = (x.to(DEV) for x in inputs)
    out, lse = torch.empty_like(q), torch.empty(T, hq, dtype=torch.float32, device=DEV)
    B.dag_attn_prefill(meta, q, k, v, out, lse)
    ws = torch.empty(B.dag_prefill_bwd_workspace_bytes(meta, hq, hkv, d), dtype=torch.uint8, device=DEV)
    names = launched_kernels(lambda: B.dag_attn_prefill_bwd(meta, q, k, v, out, dout, lse, *grads, workspace=ws))
    assert sum("k_dq_sum" in x for x in names) == pieces, names
    assert any(("k_nodes_dq2ILb%d" if d == 128 else "k_nodes64_dqILb%d") % pieces in x for x in names), names
    _check_against_oracle(dag_list, inputs, grads)


# one head a group on nodes of 16 to 32 tokens: query chunks where the items are few, or the sequences long; else the block map's tiles
@pytest.mark.parametrize("n_seqs,n_nodes,avg,hkv,chunks", [(11, 30, 22, 8, False), (4, 30, 22, 8, True), (6, 60, 22, 8, True), (11, 30, 36, 8, True), (11, 30, 22, 7, True)])
def test_single_heads_on_short_nodes(n_seqs, n_nodes, avg, hkv, chunks):
    d = 128
    rng = np.random.Generator(np.random.PCG64(8800))
    dag_list = [dags.random_dag(rng, n_nodes=n_nodes, depth=4, len_lo=avg - 9, len_hi=avg + 9)[:2] for _ in range(n_seqs)]
    T, nodes = sum(int(np.sum(L)) for L, _ in dag_list), n_seqs * n_nodes
    assert T >= 16 * nodes and chunks == (T >= 32 * nodes or T >= 1000 * n_seqs or nodes * hkv < 2560)
    inputs, grads = _forward_backward(dag_list, hkv, hkv, d, 8900)
    _, meta = build_meta(dag_list, hkv, hkv, d, torch.bfloat16)
    q, k, v, dout = (x.to(DEV) for x in inputs)
    out, lse = torch.empty_like(q), torch.empty(T, hkv, dtype=torch.float32, device=DEV)
    B.dag_attn_prefill(meta, q, k, v, out, lse)
    ws = torch.empty(B.dag_prefill_bwd_workspace_bytes(meta, hkv, hkv, d), dtype=torch.uint8, device=DEV)
    names = launched_kernels(lambda: B.dag_attn_prefill_bwd(meta, q, k, v, out, dout, lse, *grads, workspace=ws))
    assert any(("k_nodes_dq2" if chunks else "k_bwd_dq2") in x for x in names), names
    _check_against_oracle(dag_list, inputs, grads)
